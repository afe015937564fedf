// Scalar (non-MFMA) kernels for the two contractions of the pass, for any storage type and head
// dimension: what impl = GENERIC runs, which cross-checks the matrix-core kernels in the tests.  AUTO
// takes the votes kernel behind gemm.hip's logits for wide pooling windows, the edges of a single source
// and the key norms from here.  fp32 fused multiply-adds, fp32 accumulation.
#include "common.hpp"
#include "kernels.hpp"

namespace gkv {

// dot(a, b) and, optionally, |b|^2 over d elements; d is a multiple of the
// 16-byte vector width.  a comes from LDS (already widened), b from global.
template <typename T>
__device__ __forceinline__ float dot_row(const float *__restrict__ a_f32, const T *__restrict__ b,
                                         int d, float *b_sq)
{
    constexpr int V = Elem<T>::kPerVec;
    const uint4 *bv = reinterpret_cast<const uint4 *>(b);
    float acc = 0.f, sq = 0.f;
    for (int c = 0; c < d / V; ++c) {
        float t[V];
        Elem<T>::unpack(bv[c], t);
#pragma unroll
        for (int u = 0; u < V; ++u) {
            acc = fmaf(a_f32[c * V + u], t[u], acc);
            sq = fmaf(t[u], t[u], sq);
        }
    }
    if (b_sq) *b_sq = sq;
    return acc;
}

// One workgroup per query row (q, r): logits over the visible keys, then the
// row's max and sum of exp.  Stage I, softmax statistics.
template <typename T>
__global__ __launch_bounds__(256) void generic_logits_kernel(
    const T *__restrict__ Kc, const T *__restrict__ Qw, int G, int d, int N, int w, float scale,
    float *__restrict__ logits, float *__restrict__ row_max, float *__restrict__ row_sum)
{
    __shared__ float q_f32[512];
    __shared__ float red[16];
    const int row = blockIdx.x;            // q * w + r
    const int q = row / w, r = row % w, h = q / G;
    const int P = N - w, visible = P + r + 1;
    for (int c = threadIdx.x; c < d; c += 256) {
        float t;
        if constexpr (sizeof(T) == 4) t = Qw[(long)row * d + c];
        else t = bf16_to_f32(Qw[(long)row * d + c]);
        q_f32[c] = t;
    }
    __syncthreads();
    const T *kh = Kc + (long)h * N * d;
    float *lrow = logits + (long)row * N;
    float mx = -INFINITY;
    for (int j = threadIdx.x; j < visible; j += 256) {
        const float l = dot_row<T>(q_f32, kh + (long)j * d, d, nullptr) * scale;
        lrow[j] = l;
        mx = fmaxf(mx, l);
    }
    mx = block_max(mx, red);
    float z = 0.f;
    for (int j = threadIdx.x; j < visible; j += 256) z += expf(lrow[j] - mx);
    z = block_sum(z, red);
    if (threadIdx.x == 0) { row_max[row] = mx; row_sum[row] = z; }
}

// votes[q, j] = sum over window rows r of exp(l_rj - max_r) / sum_r, j < P.  A row of logits has `pitch`
// entries, the statistics of consecutive rows are `step` apart.
__global__ __launch_bounds__(256) void generic_votes_kernel(
    const float *__restrict__ logits, int pitch, const float *__restrict__ row_max,
    const float *__restrict__ row_sum, int step, int P, int w, float *__restrict__ votes)
{
    const int q = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= P) return;
    float acc = 0.f;
    for (int r = 0; r < w; ++r) {
        const int row = q * w + r;
        acc += expf(logits[(long)row * pitch + j] - row_max[(long)row * step]) / row_sum[(long)row * step];
    }
    votes[(long)q * P + j] = acc;
}

// Eq. 1 for source a of head h against prefix key j.  The source itself gets
// -inf so that it can never be its own neighbour (Eq. 3: j != i).
template <typename T>
__global__ __launch_bounds__(256) void generic_cosine_kernel(
    const T *__restrict__ Ac, const T *__restrict__ Kc, int d, int N, int P, int S,
    const int32_t *__restrict__ src, float *__restrict__ E)
{
    __shared__ float s_f32[512];
    const int a = blockIdx.y, h = blockIdx.z;
    const int i = src[h * S + a];
    const T *kh = Kc + (long)h * N * d, *ah = Ac + (long)h * N * d;   // source rows come from Ac
    float part = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) {
        float t;
        if constexpr (sizeof(T) == 4) t = ah[(long)i * d + c];
        else t = bf16_to_f32(ah[(long)i * d + c]);
        s_f32[c] = t;
    }
    __syncthreads();
    // |k_i|^2 in a fixed order (every thread computes the same sum)
    for (int c = 0; c < d; ++c) part = fmaf(s_f32[c], s_f32[c], part);
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= P) return;
    float sq;
    const float dot = dot_row<T>(s_f32, kh + (long)j * d, d, &sq);
    float e;
    if (j == i) e = -INFINITY;
    else if (part == 0.f || sq == 0.f) e = 0.f;
    else e = dot * (1.0f / sqrtf(part)) * (1.0f / sqrtf(sq));
    E[((long)h * S + a) * P + j] = e;
}

// Sum over aligned groups of LPR lanes, the same bits in every lane of a group: neighbours,
// pairs, the mirrored half row and row (data-parallel primitives), then the other row and the
// other half of the wave.
template <int LPR>
__device__ __forceinline__ float lane_group_sum(float v)
{
    static_assert(LPR == 8 || LPR == 16 || LPR == 32 || LPR == 64, "");
#define GKV_DPP(ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true))
    v += GKV_DPP(0xb1);    // quad_perm: lane ^ 1
    v += GKV_DPP(0x4e);    // quad_perm: lane ^ 2
    v += GKV_DPP(0x141);   // row_half_mirror: the other four lanes of eight
    if (LPR >= 16) v += GKV_DPP(0x140);   // row_mirror: the other eight lanes of the row
#undef GKV_DPP
    if (LPR >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if (LPR >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

// scores[h, j] = -|k_j|.  Bound by the read of the keys.  LPR lanes share a row (the smallest of
// 8, 16, 32, 64 that covers its 16-byte pieces), so that a wave's load instruction covers whole
// consecutive rows; eight loads are in flight per lane.  A wave takes 64 rows: the lane that ends
// up with row r of them stores it, one coalesced store per wave.  (A thread per row, as before,
// touches 64 rows per load instruction: 523 us for 524 MB of bf16 keys with d = 128, 1.0 TB/s;
// this way 124 us, 4.2 TB/s.)
template <typename T, int LPR, bool ONCE>
__global__ __launch_bounds__(256) void knorm_kernel(const T *__restrict__ Kc, int d, int N, int P,
                                                    float *__restrict__ scores)
{
    constexpr int V = Elem<T>::kPerVec, RPS = kWave / LPR, B = 8;   // rows per load instruction, loads in flight
    const int h = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j0 = blockIdx.x * 256 + wv * kWave;
    if (j0 >= P) return;
    const int g = lane / LPR, c = lane % LPR, vpr = d / V;
    const u32x4 *kh = reinterpret_cast<const u32x4 *>(Kc + (long)h * N * d);
    float mine = 0.f;
#pragma unroll
    for (int b0 = 0; b0 < LPR; b0 += B) {
        float sq[B];
#pragma unroll
        for (int u = 0; u < B; ++u) sq[u] = 0.f;
        for (int c0 = 0; c0 < vpr; c0 += LPR) {   // (one turn unless a row has more than 64 pieces)
            const bool in = c0 + c < vpr;
            uint4 v[B];
#pragma unroll
            for (int u = 0; u < B; ++u)
            {
                const u32x4 *p = kh + (long)min(j0 + (b0 + u) * RPS + g, P - 1) * vpr + (in ? c0 + c : 0);
                const u32x4 x = ONCE ? __builtin_nontemporal_load(p) : *p;
                v[u] = make_uint4(x.x, x.y, x.z, x.w);
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                float t[V];
                Elem<T>::unpack(v[u], t);
#pragma unroll
                for (int e = 0; e < V; ++e) sq[u] = in ? fmaf(t[e], t[e], sq[u]) : sq[u];
            }
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const float s = lane_group_sum<LPR>(sq[u]);
            mine = c == b0 + u ? s : mine;
        }
    }
    const int j = j0 + c * RPS + g;
    if (j < P) scores[(long)h * P + j] = -sqrtf(mine);
}

template <typename T>
static void launch_knorm_t(const T *Kc, int Hkv, int d, int N, int P, float *scores, hipStream_t st)
{
    const int vpr = d / Elem<T>::kPerVec;
    const dim3 grid((P + 255) / 256, Hkv);
    const bool once = reads_past_caches((size_t)Hkv * N * d * sizeof(T));
#define GKV_KNORM(LPR)                                                                                             \
    hipLaunchKernelGGL((once ? knorm_kernel<T, LPR, true> : knorm_kernel<T, LPR, false>), grid, dim3(256), 0, st, Kc, d, \
                       N, P, scores)
    if (vpr <= 8) GKV_KNORM(8);
    else if (vpr <= 16) GKV_KNORM(16);
    else if (vpr <= 32) GKV_KNORM(32);
    else GKV_KNORM(64);
#undef GKV_KNORM
}

hipError_t launch_generic_logits(const void *Kc, const void *Qw, int dtype, int Hkv, int Hq, int d,
                                 int N, int w, float scale, float *logits, float *row_max,
                                 float *row_sum, hipStream_t st)
{
    const int G = Hq / Hkv;
    if (dtype == 0)
        hipLaunchKernelGGL(generic_logits_kernel<float>, dim3(Hq * w), dim3(256), 0, st,
                           (const float *)Kc, (const float *)Qw, G, d, N, w, scale, logits, row_max,
                           row_sum);
    else
        hipLaunchKernelGGL(generic_logits_kernel<uint16_t>, dim3(Hq * w), dim3(256), 0, st,
                           (const uint16_t *)Kc, (const uint16_t *)Qw, G, d, N, w, scale, logits,
                           row_max, row_sum);
    return hipGetLastError();
}

hipError_t launch_generic_votes(const float *logits, int pitch, const float *row_max, const float *row_sum, int step,
                                int Hq, int P, int w, float *votes, hipStream_t st)
{
    hipLaunchKernelGGL(generic_votes_kernel, dim3((P + 255) / 256, Hq), dim3(256), 0, st, logits, pitch, row_max,
                       row_sum, step, P, w, votes);
    return hipGetLastError();
}

hipError_t launch_generic_cosine(const void *Ac, const void *Kc, int dtype, int Hkv, int d, int N, int P, int S,
                                 const int32_t *src, float *E, hipStream_t st)
{
    dim3 grid((P + 255) / 256, S, Hkv);
    if (dtype == 0)
        hipLaunchKernelGGL(generic_cosine_kernel<float>, grid, dim3(256), 0, st, (const float *)Ac,
                           (const float *)Kc, d, N, P, S, src, E);
    else
        hipLaunchKernelGGL(generic_cosine_kernel<uint16_t>, grid, dim3(256), 0, st,
                           (const uint16_t *)Ac, (const uint16_t *)Kc, d, N, P, S, src, E);
    return hipGetLastError();
}

hipError_t launch_knorm(const void *Kc, int dtype, int Hkv, int d, int N, int P, float *scores,
                        hipStream_t st)
{
    if (dtype == 0) launch_knorm_t((const float *)Kc, Hkv, d, N, P, scores, st);
    else launch_knorm_t((const uint16_t *)Kc, Hkv, d, N, P, scores, st);
    return hipGetLastError();
}

}  // namespace gkv
