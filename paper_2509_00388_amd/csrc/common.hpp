// Device-side helpers shared by the GraphKV kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gkv {

constexpr int kWave = 64;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes, a plain vector register group

// Per-layer quantities of a batched call, passed to kernels by value.  A batch is
// a run of layers whose tensors are contiguous ([L, H, ...]), so every (layer,
// head) pair is simply head q = l * H + h of a layer with L*H heads; only the
// budget, and with it the place of a layer's rows in the packed outputs, varies.
constexpr int kMaxLayers = 64;
struct LayerPlan {
    int32_t heads_per_layer;          // H
    int32_t budget[kMaxLayers];       // B_l
    int64_t row_off[kMaxLayers];      // H * sum_{l' < l} B_l': first output row of layer l
};

// bfloat16 <-> float: bf16 is the upper half of an IEEE float, widening is exact.
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bf16lo_to_f32(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kPerVec = 4;  // elements in a 16-byte vector
    __device__ static __forceinline__ void unpack(const uint4 &v, float *o) {
        o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y);
        o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
    }
};
template <> struct Elem<uint16_t> {
    static constexpr int kPerVec = 8;
    __device__ static __forceinline__ void unpack(const uint4 &v, float *o) {
        o[0] = bf16lo_to_f32(v.x); o[1] = bf16hi_to_f32(v.x);
        o[2] = bf16lo_to_f32(v.y); o[3] = bf16hi_to_f32(v.y);
        o[4] = bf16lo_to_f32(v.z); o[5] = bf16hi_to_f32(v.z);
        o[6] = bf16lo_to_f32(v.w); o[7] = bf16hi_to_f32(v.w);
    }
};

// Order-preserving map float -> uint32 (larger float <=> larger key).  -0.0 is
// folded onto +0.0 first so that the two compare equal, as they do as numbers.
__device__ __forceinline__ uint32_t ord_key(float f) {
    f = f + 0.0f;
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}
// Fixed butterfly order: the same inputs always give the same bits.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Block-wide reductions for blocks of up to 1024 threads; `red` holds >= 16 floats.
__device__ __forceinline__ float block_max(float v, float *red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float r = red[0];
    for (int i = 1; i < nw; ++i) r = fmaxf(r, red[i]);
    return r;
}
__device__ __forceinline__ float block_sum(float v, float *red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    float r = red[0];
    for (int i = 1; i < nw; ++i) r += red[i];
    return r;
}

// ---- wave-wide scans and reductions on the vector ALU --------------------------------
// gfx9 data-parallel primitives move a value along the lanes inside a vector instruction
// (a shift within a row of 16 lanes, then the last lane of a row to the next row, then lane 31 to
// the upper half).  A step costs a few clocks; __shfl goes through the LDS crossbar and costs
// over a hundred, which is what the one-workgroup-per-head kernels spent much of their time on.
// Lanes without a source read `identity`.
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan_op(uint32_t v, uint32_t identity, Op op)
{
#define GKV_DPP(ctrl, rows) (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, ctrl, rows, 0xf, false)
    v = op(v, GKV_DPP(0x111, 0xf));   // row_shr:1
    v = op(v, GKV_DPP(0x112, 0xf));   // row_shr:2
    v = op(v, GKV_DPP(0x114, 0xf));   // row_shr:4
    v = op(v, GKV_DPP(0x118, 0xf));   // row_shr:8
    v = op(v, GKV_DPP(0x142, 0xa));   // row_bcast:15 into rows 1 and 3
    v = op(v, GKV_DPP(0x143, 0xc));   // row_bcast:31 into rows 2 and 3
#undef GKV_DPP
    return v;
}
// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v)
{
    return wave_scan_op(v, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
// The same value in every lane (a scalar).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = wave_scan_op(v, 0xffffffffu, [](uint32_t a, uint32_t b) { return min(a, b); });
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = wave_scan_op(v, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(v), 63);
}
// LDS words that other lanes of the wave wrote before it are read after it: a wave's LDS operations complete in
// order, so it costs nothing, but without the fence the compiler may move them.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// Number of lanes below this one whose bit is set in a wave vote.
__device__ __forceinline__ uint32_t votes_below(uint64_t votes)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(votes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)votes, 0u));
}

// Exclusive sum over the threads of a workgroup of NW <= 16 waves; `total` gets the sum of all.
// `part` holds NW words of LDS that nobody else touches; contains one barrier, and the caller puts
// another between two uses of the same `part`.
template <int NW>
__device__ __forceinline__ uint32_t block_scan_add(uint32_t v, uint32_t *part, int lane, int wv, uint32_t &total)
{
    static_assert(NW <= 16, "one DPP row holds the wave sums");
    const uint32_t incl = wave_scan_add(v);
    if (lane == kWave - 1) part[wv] = incl;
    __syncthreads();
    const uint32_t sums = wave_scan_add(lane < NW ? part[lane] : 0u);
    total = (uint32_t)__builtin_amdgcn_readlane((int)sums, 63);
    // (wv is the same in all lanes of a wave: moved to a scalar so that the read below is one)
    const int w = __builtin_amdgcn_readfirstlane(wv);
    const uint32_t before = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)sums, w - 1) : 0u;
    return before + incl - v;
}

// The bin of a 2 * BLOCK-bin LDS histogram in which the count from the top reaches `need` (the
// bins hold at least `need` entries).  Thread t owns two bins, the highest pair first, so every
// thread reads eight consecutive bytes.  out[0] = the bin, out[1] = need minus the entries in
// higher bins, out[2] = entries in the bin.  Two barriers; the histogram is read before the second.
template <int BLOCK>
__device__ __forceinline__ void find_bin_block(const uint32_t *hist, uint32_t need, uint32_t *part, uint32_t *out,
                                               int tid, int lane, int wv)
{
    const int hi = 2 * (BLOCK - 1 - tid);
    const uint2 c = *reinterpret_cast<const uint2 *>(hist + hi);   // bins hi, hi + 1
    uint32_t total;
    const uint32_t above = block_scan_add<BLOCK / kWave>(c.x + c.y, part, lane, wv, total);
    if (above < need && need <= above + c.x + c.y) {
        const bool top = above + c.y >= need;
        out[0] = (uint32_t)(top ? hi + 1 : hi);
        out[1] = need - (top ? above : above + c.y);
        out[2] = top ? c.y : c.x;
    }
    __syncthreads();
}

// The m-th largest of the keys in the first NIT registers of every lane, or a value that no other keys reach (unused registers
// hold 0, below every key), all between kmin and kmax: built bit by bit from the top; the
// count of the keys that reach a trial value is one wave vote per register.  Straight-line
// code for a given NIT: branches between the votes would cost more than the votes.  A trial that exactly m keys
// reach ends it: the same keys reach it as reach the m-th largest.
template <int NIT, int R>
__device__ __forceinline__ uint32_t mth_largest_key(const uint32_t (&E)[R], uint32_t kmin, uint32_t kmax, int m)
{
    static_assert(NIT <= R, "");
    uint32_t tau = kmin;
    if (kmax > kmin) {
        for (int b = 31 - __clz(kmax - kmin); b >= 0; --b) {
            const uint32_t trial = tau + (1u << b);   // bits below b of tau - kmin are still 0
            int reach = 0;
#pragma unroll
            for (int it = 0; it < NIT; ++it) reach += (int)__popcll(__ballot(E[it] >= trial));
            if (trial > tau && reach >= m) {   // (a trial that wrapped around is beyond every key)
                tau = trial;
                if (reach == m) break;
            }
        }
    }
    return tau;
}

}  // namespace gkv
