// The two contractions of the pass on the matrix cores for any storage type and head dimension
// (fp32, and bf16 with d other than 128 or query rows that do not fill the blocks of
// mfma_score.hip).  fp32 inputs go through v_mfma_f32_32x32x2_f32, bf16 through
// v_mfma_f32_32x32x16_bf16; both accumulate in fp32.
//
// A workgroup of four waves multiplies a tile of keys with up to 128 rows (window queries, or source
// keys).  Rows and keys pass through LDS in pieces of 256 bytes a row, read from memory with coalesced
// 16-byte loads and padded by 16 bytes against bank conflicts.  A lane reads 16 bytes of its row per
// step: for bf16 the eight elements of one instruction, for fp32 four elements that feed four
// instructions (instruction e takes element e of both half-waves: k = 8 s + e and 8 s + 4 + e, the same
// pairs for rows and keys).  What bounds the kernels at these sizes is the matrix rate for fp32 and
// latency for bf16.  (A scalar kernel with a workgroup per query row, each re-reading all keys: 234 us
// for 1024 rows x 4096 fp32 keys with d = 128, 4.6 TFLOP/s; this way 23 us, 47 TFLOP/s.)
#include "common.hpp"
#include "kernels.hpp"

namespace gkv {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float acc16 __attribute__((ext_vector_type(16)));

// PB: bytes of a row staged at a time, 256 or, for rows of up to 128 bytes, 128 (half the loads and LDS writes would
// be of zeros otherwise).
constexpr int pitch_of(int PB) { return PB + 16; }   // in LDS

__device__ __forceinline__ int mfma_row(int i, int hh) { return 8 * (i >> 2) + 4 * hh + (i & 3); }

// acc += (32 rows of a) x (32 rows of b)^T over one step (32 bytes of every row).
template <typename T> __device__ __forceinline__ void mfma_step(const uint4 &a, const uint4 &b, acc16 &acc);
template <> __device__ __forceinline__ void mfma_step<float>(const uint4 &a, const uint4 &b, acc16 &acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ void mfma_step<uint16_t>(const uint4 &a, const uint4 &b, acc16 &acc)
{
    union { uint4 u; bf16x8_t v; } x{a}, y{b};
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, y.v, acc, 0, 0, 0);
}

template <typename T> __device__ __forceinline__ float sum_squares(const uint4 &v, float s)
{
    float t[Elem<T>::kPerVec];
    Elem<T>::unpack(v, t);
#pragma unroll
    for (int e = 0; e < Elem<T>::kPerVec; ++e) s = fmaf(t[e], t[e], s);
    return s;
}

// ROWS rows on their way to the LDS: bytes c0 .. c0 + PB - 1 of each (row(r) = address of row r), zeros past the end
// of a row.  The loads of a piece are asked for while the piece before it is multiplied.  (Before, each piece was
// fetched four loads at a time behind the barrier that frees the LDS, 256 bytes whatever the row: logits and edges of
// 16 heads x 8160 bf16 keys of 64 with 32 rows 14.1 and 14.9 us, 11.3 and 12.4 this way; edges of 8 heads x 4064
// fp32 keys of 128 with 32 sources 12.2, now 10.7.)
template <int ROWS, int PB> struct Staged {
    static constexpr int PIECES = PB / 16, PER = ROWS * PIECES / 256;
    static_assert(ROWS * PIECES % 256 == 0, "pieces per thread");
    uint4 v[PER];
    template <typename Row> __device__ __forceinline__ void ask(int c0, int row_bytes, int tid, Row &&row)
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int g = tid + u * 256;
            v[u] = *reinterpret_cast<const uint4 *>(row(g / PIECES) + min(c0 + 16 * (g % PIECES), row_bytes - 16));
        }
    }
    __device__ __forceinline__ void put(unsigned char *lds, int c0, int row_bytes, int tid) const
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int g = tid + u * 256;
            const bool in = c0 + 16 * (g % PIECES) < row_bytes;
            *reinterpret_cast<uint4 *>(lds + (g / PIECES) * pitch_of(PB) + 16 * (g % PIECES)) = in ? v[u] : make_uint4(0, 0, 0, 0);
        }
    }
};

__device__ __forceinline__ float other_half(float x)   // x of the lane 32 places away
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

// (m, z) <- merge with (m2, z2): running maximum and sum of exp(l - maximum).
__device__ __forceinline__ void merge_exp(float &m, float &z, float m2, float z2)
{
    const float mn = fmaxf(m, m2);
    z = mn == -INFINITY ? 0.f : z * expf(m - mn) + z2 * expf(m2 - mn);
    m = mn;
}

// Waves of a workgroup: RS row groups x (4 / RS) key streams of 32 keys; NBR blocks of 32 rows.
template <int NBR> struct Shape {
    static constexpr int RS = NBR >= 2 ? 2 : 1, STREAMS = 4 / RS, NBW = NBR / RS, TR = 32 * NBR, TK = 32 * STREAMS;
};

// Stage I, logits of the window queries (scaled; `pitch` of the N to a row, the P prefix keys' at least) and per
// (chunk of keys, row) the maximum and the sum of exp over the chunk's visible keys.  Keys are the rows of the products, queries the
// columns: a lane owns one query and keeps its statistics without cross-lane traffic.  MANY: a workgroup takes
// `per_wg` consecutive chunks, whole tiles each, and keeps their statistics apart.
// (Three waves per SIMD at least: 8 heads x 8192 fp32 keys of 128 with 128 rows 55.3 -> 54.4 us for the scores,
// with 256 rows 91.6 -> 90.4.)
template <typename T, int NBR, int PB, bool MANY>
__global__ __launch_bounds__(256, 3) void gemm_logits_kernel(
    const T *__restrict__ Kc, const T *__restrict__ Qw, int d, int N, int P, int w, int R, float scale,
    int chunk_keys, int nchunks, int per_wg, int pitch, float *__restrict__ logits, float *__restrict__ part)
{
    using Sh = Shape<NBR>;
    constexpr int PITCH = pitch_of(PB), STEPS = PB / 32;
    __shared__ __align__(16) unsigned char kt[Sh::TK * PITCH], qt[Sh::TR * PITCH];
    __shared__ float sm[Sh::STREAMS][Sh::TR], sz[Sh::STREAMS][Sh::TR];
    const int h = blockIdx.y, row0 = blockIdx.z * Sh::TR;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv % Sh::STREAMS, rs = wv / Sh::STREAMS;
    const int row_bytes = d * (int)sizeof(T);
    const char *Kh = reinterpret_cast<const char *>(Kc + (long)h * N * d);
    const char *Qh = reinterpret_cast<const char *>(Qw + (long)h * R * d);
    const int first = blockIdx.x * (MANY ? per_wg : 1), last = MANY ? min(nchunks, first + per_wg) : first + 1;
    const bool whole = row_bytes <= PB;   // (the queries stay when they fit whole)
    Staged<Sh::TK, PB> kin;
    Staged<Sh::TR, PB> qin;
    auto ask_keys = [&](int t0, int c0) {
        kin.ask(c0, row_bytes, tid, [&](int r) { return Kh + (long)min(t0 + r, N - 1) * row_bytes; });
    };
    auto ask_queries = [&](int c0) {
        qin.ask(c0, row_bytes, tid, [&](int r) { return Qh + (long)min(row0 + r, R - 1) * row_bytes; });
    };
    ask_keys(first * chunk_keys, 0);
    ask_queries(0);
    for (int chunk = first; chunk < last; ++chunk) {
        const int k0 = chunk * chunk_keys, k1 = min(N, k0 + chunk_keys), kstore = min(k1, pitch);
        float m[Sh::NBW], z[Sh::NBW];
        int last_vis[Sh::NBW];
#pragma unroll
        for (int b = 0; b < Sh::NBW; ++b) {
            m[b] = -INFINITY;
            z[b] = 0.f;
            last_vis[b] = min(P + (row0 + 32 * (rs * Sh::NBW + b) + l32) % w, k1 - 1);
        }
        for (int t0 = k0; t0 < k1; t0 += Sh::TK) {
            acc16 acc[Sh::NBW];
#pragma unroll
            for (int b = 0; b < Sh::NBW; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
            for (int c0 = 0; c0 < row_bytes; c0 += PB) {
                __syncthreads();   // the tiles in LDS are free
                kin.put(kt, c0, row_bytes, tid);
                if (!whole || (t0 == k0 && chunk == first)) qin.put(qt, c0, row_bytes, tid);
                __syncthreads();
                // the next piece: of this tile, or of the next one (past the last, rows that are there)
                const int cn = c0 + PB < row_bytes ? c0 + PB : 0;
                ask_keys(cn ? t0 : t0 + Sh::TK, cn);
                if (!whole) ask_queries(cn);
                const int steps = (min(row_bytes - c0, PB) + 31) / 32;
                const unsigned char *kp = kt + (32 * stream + l32) * PITCH + 16 * hh;
                const unsigned char *qp = qt + (32 * rs * Sh::NBW + l32) * PITCH + 16 * hh;
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    if (s >= steps) break;
                    const uint4 k = *reinterpret_cast<const uint4 *>(kp + 32 * s);
#pragma unroll
                    for (int b = 0; b < Sh::NBW; ++b)
                        mfma_step<T>(k, *reinterpret_cast<const uint4 *>(qp + 32 * b * PITCH + 32 * s), acc[b]);
                }
            }
            const int key0 = t0 + 32 * stream;
#pragma unroll
            for (int b = 0; b < Sh::NBW; ++b) {
                const int row = row0 + 32 * (rs * Sh::NBW + b) + l32;
                float tm = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    acc[b][i] *= scale;
                    if (key0 + mfma_row(i, hh) <= last_vis[b]) tm = fmaxf(tm, acc[b][i]);
                }
                const float mn = fmaxf(m[b], tm);
                if (mn != -INFINITY) {
                    float zz = z[b] * expf(m[b] - mn);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (key0 + mfma_row(i, hh) <= last_vis[b]) zz += expf(acc[b][i] - mn);
                    m[b] = mn;
                    z[b] = zz;
                }
                if (row < R) {
                    float *o = logits + ((long)h * R + row) * pitch;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int key = key0 + 8 * v + 4 * hh;
                        if ((pitch & 3) == 0 && key + 3 < kstore) {
                            *reinterpret_cast<float4 *>(o + key) =
                                make_float4(acc[b][4 * v], acc[b][4 * v + 1], acc[b][4 * v + 2], acc[b][4 * v + 3]);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (key + e < kstore) o[key + e] = acc[b][4 * v + e];
                        }
                    }
                }
            }
        }
        // the half-waves (same query, other keys), then the key streams
#pragma unroll
        for (int b = 0; b < Sh::NBW; ++b) {
            merge_exp(m[b], z[b], other_half(m[b]), other_half(z[b]));
            if (hh == 0) {
                sm[stream][32 * (rs * Sh::NBW + b) + l32] = m[b];
                sz[stream][32 * (rs * Sh::NBW + b) + l32] = z[b];
            }
        }
        __syncthreads();
        if (tid < Sh::TR && row0 + tid < R) {
            float mm = sm[0][tid], zz = sz[0][tid];
#pragma unroll
            for (int u = 1; u < Sh::STREAMS; ++u) merge_exp(mm, zz, sm[u][tid], sz[u][tid]);
            float *o = part + (((long)h * nchunks + chunk) * R + row0 + tid) * 2;
            o[0] = mm;
            o[1] = zz;
        }
    }
}

// Votes, pooling and the mean over the group in one go: scores[h, j] = 1/G sum_g pool(votes of query
// head g).  A workgroup takes KEYS keys (pool_half of them on either side only for the pooling), its
// PARTS groups of KEYS threads share the query rows, each with SUMS sums per key (the order of a key's
// additions is that of PARTS * SUMS groups); the statistics of up to kVoteRows rows at a time are
// merged from the chunks into LDS first.  Average pooling adds the whole group before it pools, so only
// max pooling has to stop at every query head.  (Merging the statistics of one query head at a time:
// 24 us for 8 heads of 128 rows x 4064 keys, 30 us for 8160; this way, merge included, 17 and 27 us.)
constexpr int kVoteHalf = 32;    // widest pooling half-window taken here
constexpr int kVoteRows = 512;   // rows whose statistics sit in LDS

template <int KEYS, int PARTS, int SUMS>   // SUMS: 1 or 2
__global__ __launch_bounds__(KEYS * PARTS) void gemm_votes_kernel(
    const float *__restrict__ logits, int pitch, const float *__restrict__ part, int chunks, int P, int w, int G,
    int pool_half, int pool_mode, float *__restrict__ scores)
{
    constexpr int NT = KEYS * PARTS, GROUPS = PARTS * SUMS, U = 8 / SUMS;
    __shared__ float vs[GROUPS][KEYS], s_max[kVoteRows], s_inv[kVoteRows];
    const int h = blockIdx.y, tid = threadIdx.x, t = tid % KEYS, p = tid / KEYS;
    const int R = G * w, tile = KEYS - 2 * pool_half;
    const int j = blockIdx.x * tile - pool_half + t;          // this thread's key
    const bool in = j >= 0 && j < P;
    const int jc = min(max(j, 0), P - 1);
    const float *lh = logits + (long)h * R * pitch + jc;
    float total = 0.f, v[SUMS] = {};
    auto put_parts = [&] {
#pragma unroll
        for (int q = 0; q < SUMS; ++q) {
            vs[p + q * PARTS][t] = v[q];
            v[q] = 0.f;
        }
    };
    auto all_parts = [&] {
        float sum = vs[0][t];
#pragma unroll
        for (int u = 1; u < GROUPS; ++u) sum += vs[u][t];
        return sum;
    };
    // rows [first, last) of the head, whose statistics start at entry first - base of the tables
    auto vote = [&](int first, int last, int base) {
        auto add = [&](int r, float &sum) { sum += expf(lh[(long)r * pitch] - s_max[r - base]) * s_inv[r - base]; };
        int r = first + p;
        if (SUMS > 1) {
#pragma unroll U
            for (; r + (SUMS - 1) * PARTS < last; r += GROUPS)
#pragma unroll
                for (int q = 0; q < SUMS; ++q) add(r + q * PARTS, v[q]);
            if (r < last) add(r, v[0]);
        } else {
#pragma unroll U
            for (; r < last; r += PARTS) add(r, v[0]);
        }
    };
    for (int base = 0; base < R; base += kVoteRows) {
        const int rows = min(kVoteRows, R - base);
        __syncthreads();
        // the chunks of a row are merged by 8 to 64 lanes, as many as there are for all rows at once
        int per_row = 64;
        while (per_row > 8 && NT / per_row < rows) per_row >>= 1;
        for (int r0 = 0; r0 < rows; r0 += NT / per_row) {
            const int r = r0 + tid / per_row, sub = tid & (per_row - 1);
            float mm = -INFINITY, zz = 0.f;
            if (r < rows)
                for (int c0 = sub; c0 < chunks; c0 += 4 * per_row) {   // (four loads leave together)
                    float2 o[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        o[u] = *reinterpret_cast<const float2 *>(
                            part + (((long)h * chunks + min(c0 + per_row * u, chunks - 1)) * R + base + r) * 2);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (c0 + per_row * u < chunks) merge_exp(mm, zz, o[u].x, o[u].y);
                }
            for (int o = per_row >> 1; o > 0; o >>= 1) {
                const float m2 = __shfl_xor(mm, o, kWave), z2 = __shfl_xor(zz, o, kWave);
                merge_exp(mm, zz, m2, z2);
            }
            if (sub == 0 && r < rows) {
                s_max[r] = mm;
                s_inv[r] = 1.0f / zz;
            }
        }
        __syncthreads();
        if (pool_mode == 0) {
            vote(base, base + rows, base);
            continue;
        }
        // max pooling: the rows of the query heads this batch touches, one head after the other
        for (int g = base / w; g <= (base + rows - 1) / w; ++g) {
            vote(max(base, g * w), min(base + rows, (g + 1) * w), base);
            if ((g + 1) * w > base + rows) break;   // the head goes on in the next batch
            put_parts();
            __syncthreads();
            const float sum = all_parts();
            __syncthreads();
            if (p == 0) vs[0][t] = in ? sum : -INFINITY;
            __syncthreads();
            if (p == 0 && t >= pool_half && t < KEYS - pool_half) {
                float best = -INFINITY;
                for (int u = t - pool_half; u <= t + pool_half; ++u) best = fmaxf(best, vs[0][u]);
                total += best;
            }
            __syncthreads();
        }
    }
    if (pool_mode == 0) {
        put_parts();
        __syncthreads();
        const float sum = all_parts();
        __syncthreads();
        if (p == 0) vs[0][t] = in ? sum : 0.f;      // zero padding outside the row
        __syncthreads();
        if (p == 0 && t >= pool_half && t < KEYS - pool_half) {
            for (int u = t - pool_half; u <= t + pool_half; ++u) total += vs[0][u];
            total = total / (float)(2 * pool_half + 1);
        }
    }
    if (p == 0 && in && t >= pool_half && t < KEYS - pool_half) scores[(long)h * P + j] = total / (float)G;
}

// Row statistics on their own: stat [rows] (max, sum).  Every workgroup of the votes kernel would otherwise
// merge all chunks of its head again, which with 64 chunks takes longer than the votes.  16 lanes per row.
__global__ __launch_bounds__(256) void merge_rows_kernel(const float *__restrict__ part, int chunks, int R, int rows,
                                                         float2 *__restrict__ stat)
{
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;
    const int h = min(row, rows - 1) / R, r = min(row, rows - 1) % R;
    float m = -INFINITY, z = 0.f;
    for (int c0 = sub; c0 < chunks; c0 += 64) {   // (four loads leave together)
        float2 o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            o[u] = *reinterpret_cast<const float2 *>(part + (((long)h * chunks + min(c0 + 16 * u, chunks - 1)) * R + r) * 2);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + 16 * u < chunks) merge_exp(m, z, o[u].x, o[u].y);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(m, o, kWave), z2 = __shfl_xor(z, o, kWave);
        merge_exp(m, z, m2, z2);
    }
    if (sub == 0 && row < rows) stat[row] = make_float2(m, z);
}

// Eq. 1: E[h, a, j] = cosine of row src[h, a] of Ac and row j of Kc, -inf where j is the source itself
// (Eq. 3).  Sources are the rows of the products and keys the columns: a lane owns one key, whose norm
// it sums from the very registers that feed the products, and stores run along the keys.
// (Two waves per SIMD at least, which prefetched pieces of 256 bytes and four row blocks would otherwise exceed by ten
// registers: 8 heads x 8160 bf16 keys of 256 with 128 sources, key norms, whole call 93.6 us, 79.7 this way, 78.5 with
// nothing prefetched; 96 sources 83.4, 69.3 and 72.3; 32 heads with 128 205, 164 and 176.  The sources' norms, a thread each
// while the others wait, one LDS read behind the other: edges of 8 heads x 4064 fp32 keys with 32 sources 11.5 us, four at a
// time 9.9.)
template <typename T, int NBR, int PB>
__global__ __launch_bounds__(256, 2) void gemm_cosine_kernel(
    const T *__restrict__ Ac, const T *__restrict__ Kc, int d, int N, int P, int S, const int32_t *__restrict__ src,
    int chunk_keys, float *__restrict__ E)
{
    using Sh = Shape<NBR>;
    constexpr int PITCH = pitch_of(PB), STEPS = PB / 32;
    __shared__ __align__(16) unsigned char kt[Sh::TK * PITCH], qt[Sh::TR * PITCH];
    __shared__ float inv_s[Sh::TR];
    __shared__ int32_t idx_s[Sh::TR];
    const int h = blockIdx.y, row0 = blockIdx.z * Sh::TR;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv % Sh::STREAMS, rs = wv / Sh::STREAMS;
    const int row_bytes = d * (int)sizeof(T);
    const char *Kh = reinterpret_cast<const char *>(Kc + (long)h * N * d);
    const char *Ah = reinterpret_cast<const char *>(Ac + (long)h * N * d);
    const int k0 = blockIdx.x * chunk_keys, k1 = min(P, k0 + chunk_keys);
    const bool whole = row_bytes <= PB;
    Staged<Sh::TK, PB> kin;
    Staged<Sh::TR, PB> qin;
    auto ask_keys = [&](int t0, int c0) {
        kin.ask(c0, row_bytes, tid, [&](int r) { return Kh + (long)min(t0 + r, P - 1) * row_bytes; });
    };
    auto ask_sources = [&](int c0) {
        qin.ask(c0, row_bytes, tid, [&](int r) { return Ah + (long)idx_s[r] * row_bytes; });
    };
    const int32_t mine = src[(long)h * S + min(row0 + tid, S - 1)];   // (in front of the keys: the sources' rows wait for it)
    ask_keys(k0, 0);
    if (tid < Sh::TR) idx_s[tid] = mine;
    __syncthreads();
    ask_sources(0);
    for (int t0 = k0; t0 < k1; t0 += Sh::TK) {
        acc16 acc[Sh::NBW];
#pragma unroll
        for (int b = 0; b < Sh::NBW; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
        float sq = 0.f, sq_src = 0.f;
        for (int c0 = 0; c0 < row_bytes; c0 += PB) {
            __syncthreads();   // the tiles in LDS are free
            kin.put(kt, c0, row_bytes, tid);
            if (!whole || t0 == k0) qin.put(qt, c0, row_bytes, tid);
            __syncthreads();
            const int cn = c0 + PB < row_bytes ? c0 + PB : 0;   // the next piece
            ask_keys(cn ? t0 : t0 + Sh::TK, cn);
            if (!whole) ask_sources(cn);
            const int steps = (min(row_bytes - c0, PB) + 31) / 32;
            if (t0 == k0 && tid < Sh::TR) {   // a thread per source (zeros behind the row's end), four reads at a time
#pragma unroll
                for (int u0 = 0; u0 < 2 * STEPS; u0 += 4) {
                    uint4 x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const uint4 *>(qt + tid * PITCH + 16 * (u0 + u));
#pragma unroll
                    for (int u = 0; u < 4; ++u) sq_src = sum_squares<T>(x[u], sq_src);
                }
            }
            const unsigned char *kp = kt + (32 * stream + l32) * PITCH + 16 * hh;
            const unsigned char *qp = qt + (32 * rs * Sh::NBW + l32) * PITCH + 16 * hh;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (s >= steps) break;
                const uint4 k = *reinterpret_cast<const uint4 *>(kp + 32 * s);
                sq = sum_squares<T>(k, sq);
#pragma unroll
                for (int b = 0; b < Sh::NBW; ++b)
                    mfma_step<T>(*reinterpret_cast<const uint4 *>(qp + 32 * b * PITCH + 32 * s), k, acc[b]);
            }
        }
        if (t0 == k0) {
            if (tid < Sh::TR) inv_s[tid] = sq_src == 0.f ? 0.f : 1.0f / sqrtf(sq_src);
            __syncthreads();
        }
        sq += other_half(sq);
        const float inv_k = sq == 0.f ? 0.f : 1.0f / sqrtf(sq);   // a zero key or source: all edges 0
        const int key = t0 + 32 * stream + l32;
        if (key < k1) {
#pragma unroll
            for (int b = 0; b < Sh::NBW; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = 32 * (rs * Sh::NBW + b) + mfma_row(i, hh);
                    if (row0 + r < S)
                        E[((long)h * S + row0 + r) * P + key] =
                            key == idx_s[r] ? -INFINITY : acc[b][i] * inv_s[r] * inv_k;
                }
        }
    }
}

// Rows per workgroup: up to 128, no more than the rows need.
int row_blocks(int rows) { return rows <= 32 ? 1 : (rows <= 64 ? 2 : 4); }

// Keys per workgroup: whole key tiles (128 keys with one row block, 64 with more), for up to 1024 workgroups.
int gemm_chunk_keys(int Hkv, int rows, int N)
{
    const int nb = row_blocks(rows), groups = (rows + 32 * nb - 1) / (32 * nb);
    const long total = (long)Hkv * groups * N;
    long ck = (total + 1023) / 1024;
    // (with one row block a tile's products are few next to fetching the rows: two tiles a workgroup where
    // that still leaves 512 workgroups, 16 heads of 8160 keys 18.4 -> 16.2 us)
    if (nb == 1 && ck < 256) ck = total / 512 < 256 ? (total + 511) / 512 : 256;
    const long tile = nb == 1 ? Shape<1>::TK : Shape<4>::TK;
    return (int)((ck + tile - 1) / tile * tile);
}

}  // namespace

// A softmax sum depends in its last bits on where the keys are cut, so a batch cuts them as one of its layers
// alone would and gives a workgroup several chunks (whole pass, us, cut by all heads / by a layer's: 8 layers of 8
// fp32 heads x 4096 keys 262 / 267, 32 of 4 bf16 heads x 4096 with 448 rows 812 / 836, 8 x 4 x 2048 129 / 136).
// trim: keep the prefix keys' logits only, for a buffer that all of them do not fit (rows that are a power of two
// apart or not: 241 us trimmed / 249 whole for 256 rows x 32768 keys, 69 / 67 for 448 x 8192).  From 32 MiB of a
// layer's logits on there are no more chunks than hold the statistics within what the scalar kernels would need
// for their votes (4 P / w bytes a row) and the logits of the window's own keys (4 w): trimmed, this route
// then fits every buffer that route fits.
GemmScorePlan gemm_score_plan(int Hkv, int layer_heads, int G, int w, int N, bool trim)
{
    GemmScorePlan pl;
    const int rows = G * w, P = N - w;
    int ck = gemm_chunk_keys(layer_heads, rows, N);
    if ((long)layer_heads * rows * N >= (8L << 20)) {
        const int most = max(1, w / 2 + P / (2 * w) - 2), tile = row_blocks(rows) == 1 ? Shape<1>::TK : Shape<4>::TK;
        const int least = (N + most - 1) / most;
        if (ck < least) ck = (least + tile - 1) / tile * tile;
    }
    pl.chunk_keys = ck;
    pl.chunks = (N + ck - 1) / ck;
    // as many workgroups a head as the heads of the launch ask for, evenly filled
    const int all = gemm_chunk_keys(Hkv, rows, N), wgs = (N + all - 1) / all;
    pl.per_wg = max(1, (pl.chunks + wgs - 1) / wgs);
    pl.pitch = trim ? P : N;
    // (a single chunk's statistics are the rows')
    pl.part_bytes = pl.chunks > 1 ? (size_t)Hkv * rows * pl.chunks * 2 * sizeof(float) : 0;
    return pl;
}

bool gemm_votes_pools(int pool_kernel) { return (pool_kernel - 1) / 2 <= kVoteHalf; }

template <typename T>
static void launch_logits_t(const T *K, const T *Q, int Hkv, int R, int d, int N, int P, int w, float scale,
                            const GemmScorePlan &pl, float *logits, float *part, hipStream_t st)
{
    const int nb = row_blocks(R);
    const dim3 grid((pl.chunks + pl.per_wg - 1) / pl.per_wg, Hkv, (R + 32 * nb - 1) / (32 * nb));
    const bool narrow = d * (int)sizeof(T) <= 128;
#define GKV_LOGITS(NB)                                                                                             \
    do {                                                                                                           \
        auto *kernel = narrow ? (pl.per_wg > 1 ? gemm_logits_kernel<T, NB, 128, true> : gemm_logits_kernel<T, NB, 128, false>)  \
                              : (pl.per_wg > 1 ? gemm_logits_kernel<T, NB, 256, true> : gemm_logits_kernel<T, NB, 256, false>); \
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, K, Q, d, N, P, w, R, scale, pl.chunk_keys, pl.chunks,   \
                           pl.per_wg, pl.pitch, logits, part);                                                     \
    } while (0)
    if (nb == 1) GKV_LOGITS(1);
    else if (nb == 2) GKV_LOGITS(2);
    else GKV_LOGITS(4);
#undef GKV_LOGITS
}

hipError_t launch_gemm_logits(const void *Kc, const void *Qw, int dtype, int Hkv, int Hq, int d, int N, int w,
                              float scale, const GemmScorePlan &pl, float *logits, float *part, hipStream_t st)
{
    const int R = Hq / Hkv * w, P = N - w;
    if (dtype == 0) launch_logits_t((const float *)Kc, (const float *)Qw, Hkv, R, d, N, P, w, scale, pl, logits, part, st);
    else launch_logits_t((const uint16_t *)Kc, (const uint16_t *)Qw, Hkv, R, d, N, P, w, scale, pl, logits, part, st);
    return hipGetLastError();
}

// From 8192 (row, chunk) pairs a head on (us, merged by every votes workgroup / first: 128 rows x 128 chunks
// 39.7 / 26.6, 128 x 64 18.0 / 17.1, 128 x 32 14.9 / 19.4, 16 x 64 14.3 / 16.5).
bool gemm_merges_first(const GemmScorePlan &pl, int rows) { return pl.chunks > 1 && (long)pl.chunks * rows >= 8192; }

hipError_t launch_gemm_merge(const float *part, const GemmScorePlan &pl, int Hkv, int Hq, int w, float *stat,
                             hipStream_t st)
{
    const int R = Hq / Hkv * w, rows = Hq * w;
    hipLaunchKernelGGL(merge_rows_kernel, dim3((rows + 15) / 16), dim3(256), 0, st, part, pl.chunks, R, rows,
                       (float2 *)stat);
    return hipGetLastError();
}

hipError_t launch_gemm_votes(const float *logits, const GemmScorePlan &pl, const float *part, int chunks, int Hkv,
                             int layer_heads, int Hq, int N, int w, int pool_kernel, int pool_mode, float *scores,
                             hipStream_t st)
{
    const int G = Hq / Hkv, P = N - w, half = (pool_kernel - 1) / 2;
#define GKV_VOTES(KEYS, PARTS, SUMS)                                                                               \
    hipLaunchKernelGGL((gemm_votes_kernel<KEYS, PARTS, SUMS>), dim3((P + KEYS - 2 * half - 1) / (KEYS - 2 * half), Hkv), \
                       dim3(KEYS * PARTS), 0, st, logits, pl.pitch, part, chunks, P, w, G, half, pool_mode, scores)
    // few query rows: half-size workgroups; few keys: narrower ones, to reach all compute units.  The order of a
    // key's additions goes by the layer's keys, so that a batch gives the same bits.
    if (G * w <= 32) GKV_VOTES(256, 2, 1);
    else if ((long)layer_heads * P > 40000) GKV_VOTES(256, 4, 1);
    else if ((long)Hkv * P > 40000) GKV_VOTES(256, 4, 2);   // (a batch; as 128 x 8: 136 -> 144 us in the last case above)
    else GKV_VOTES(128, 8, 1);
#undef GKV_VOTES
    return hipGetLastError();
}

template <typename T>
static void launch_cosine_t(const T *A, const T *K, int Hkv, int d, int N, int P, int S, const int32_t *src, float *E,
                            hipStream_t st)
{
    const int nb = row_blocks(S), ck = gemm_chunk_keys(Hkv, S, P);
    const dim3 grid((P + ck - 1) / ck, Hkv, (S + 32 * nb - 1) / (32 * nb));
    const bool narrow = d * (int)sizeof(T) <= 128;
#define GKV_COSINE(NB)                                                                                             \
    do {                                                                                                           \
        auto *kernel = narrow ? gemm_cosine_kernel<T, NB, 128> : gemm_cosine_kernel<T, NB, 256>;                   \
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, A, K, d, N, P, S, src, ck, E);                          \
    } while (0)
    if (nb == 1) GKV_COSINE(1);
    else if (nb == 2) GKV_COSINE(2);
    else GKV_COSINE(4);
#undef GKV_COSINE
}

hipError_t launch_gemm_cosine(const void *Ac, const void *Kc, int dtype, int Hkv, int d, int N, int P, int S,
                              const int32_t *src, float *E, hipStream_t st)
{
    if (dtype == 0) launch_cosine_t((const float *)Ac, (const float *)Kc, Hkv, d, N, P, S, src, E, st);
    else launch_cosine_t((const uint16_t *)Ac, (const uint16_t *)Kc, Hkv, d, N, P, S, src, E, st);
    return hipGetLastError();
}

}  // namespace gkv
