// Eq. 1 and Eq. 3 on the matrix cores: cosine of every source key against every
// prefix key (bf16 inputs, d = 128, fp32 accumulation), and each source's m
// largest edges without ever storing the S x P edge block.
//
// Up to 96 source rows (three 32-row MFMA blocks) are held in registers; keys stream
// from HBM through the LDS into MFMA operand registers, in tiles that a workgroup
// shares as in the scoring kernels, or (the filter pass) in blocks of a wave's own.  The
// squared norm of each streamed key is accumulated from the very registers that feed
// the MFMA, so the keys are read once.
//
// Neighbourhoods in one streaming pass:
//   1. a first pass over an evenly strided sample of the keys (every 8th) takes a
//      bound for each source, a value that r of its sampled edges reach and hardly any
//      more, where r < m is chosen so that all but about one source in 10^7
//      have at least m edges above it (mfma_bound_rank; r = m would make that certain,
//      a subset's m-th largest can only be smaller, but lets 8 m keys through
//      where r lets 8 r);
//   2. the streaming pass keeps only the edges that reach the bound (a couple of
//      hundred per source), parked in LDS and appended to per-source lists;
//   3. an exact (value desc, index asc) top-m over each short list -- exact whenever
//      the list holds m entries or more, since it then holds every edge that is at
//      least the bound and the m largest are among those.
// A source whose list overflows (masses of equal edges, adversarial order) or comes
// out short of m entries sets a per-head flag and that head is redone exactly, row by
// row (redo_rows in select.hip).
//
// A neighbourhood depends on the keys alone, so a source that comes back in a later
// round keeps its list.  The first round's passes also take a third 32-row group per
// workgroup: the nodes ranked right behind the sources, which are the likeliest new
// sources of the following rounds (the decay only lowers scores, so whoever moves up
// comes from just below the cut).  Their candidate lists are kept, and a later round
// runs the exact select on them when they are promoted; only a new source without a
// kept list goes through the bound and filter passes again (a per-head count of rows
// in use; heads without such a source return at once).
#include "common.hpp"
#include "kernels.hpp"
#include "match.hpp"
#include "mfma_tile.hpp"
#include "reach.hpp"

#include <math.h>

namespace gkv {

namespace {

constexpr int kSB = 2;            // source blocks of 32 per workgroup = row groups of waves
constexpr int kRows = kSB * kBlk; // source rows per workgroup
constexpr int kThreads = 256 * kSB;

// The per-row buffers (tau, cand, cand_cnt) hold `pitch` rows per head, of which a launch's source list takes the first.
struct FilterArgs {
    const int32_t *n_src;  // [Hkv] rows of the head's source list in use; null: all S
    const float *tau;      // [Hkv, pitch] the bound pass's value per row: edges below it are dropped
    // or, with few heads, what the bound pass's chunks left (null: tau has the bounds), and its sample
    const float *part;
    int rank, key_stride;
    uint2 *cand;           // [Hkv, pitch, row_slots] (edge bits, key index): a slice of slice_cap per key chunk
    int32_t *cand_cnt;     // [Hkv, pitch, chunk_slots] entries in each slice
    int32_t *overflow;     // [Hkv]
    long row_slots;
    int chunk_slots, slice_cap;
    int sgroups;           // workgroups (groups of source rows) per key chunk
    int src_pitch;         // entries per head of the source list
    int pitch;
};

// Both kernels below: a workgroup has 4 key streams (wave & 3) and 2 source row
// groups (wave >> 2): wave (stream, g) multiplies source rows 32g .. 32g+31 of its
// 64-row group with rows 32*stream .. +31 of every key tile.  Two waves share a
// SIMD and overlap each other's MFMA and vector work.  The edge is
// e = (dot * 1/|k_j|) * 1/|k_i| in both, so the sample pass and the filter pass
// produce the same bits.

// Sources are rows of Ac, the streamed rows are rows of Kc (both [Hkv, N, 128]); for
// Eq. 1 both are the keys, the other pairings of the paper's Discussion pass two tensors.
// This wave's 32 source rows -> MFMA operand registers (slots beyond S repeat the
// last source); 1/|k_i| and the source index of the workgroup's rows go to LDS.
__device__ __forceinline__ void load_sources(const uint16_t *Ah, const int32_t *src_h, int S,
                                             int s_base, int grp, int stream, int l32, int hh,
                                             bf16x8 (&q)[kSteps], float *inv_s, int32_t *idx_s)
{
    const int slot = min(s_base + kBlk * grp + l32, S - 1);
    const int32_t i = src_h[slot];
    const uint16_t *p = Ah + (long)i * kD + 8 * hh;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) q[s] = load8(p + 16 * s);
    float sq = half_row_sumsq(q);
    sq = add_other_half(sq);
    if (stream == 0 && hh == 0) {
        inv_s[kBlk * grp + l32] = inv_norm(sq);
        idx_s[kBlk * grp + l32] = i;
    }
}

// Dense block: E[h, slot, key] = e, -inf where the key is the source itself.
__global__ __launch_bounds__(kThreads) void cosine_dense_kernel(
    const uint16_t *__restrict__ Ac, const uint16_t *__restrict__ Kc, int N, int P, int S,
    const int32_t *__restrict__ src, int chunk_cols, float *__restrict__ E)
{
    __shared__ float inv_s[kRows];
    __shared__ int32_t idx_s[kRows];
    extern __shared__ __align__(16) unsigned char smem[];   // two key tiles
    unsigned char *kt = smem;

    const int h = blockIdx.y, chunk = blockIdx.x, s_base = blockIdx.z * kRows;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv & 3, grp = wv >> 2;
    const uint16_t *Kh = Kc + (long)h * N * kD;
    const int c0 = chunk * chunk_cols, c1 = min(P, c0 + chunk_cols);
    if (c0 >= P) return;

    // (slots beyond S repeat the last source)
    bf16x8 q[1][kSteps];
    float inv_src[16];
    auto sources = [&] {
        const uint16_t *Ah = Ac + (long)h * N * kD;
        const int32_t *src_h = src + (long)h * S;
        spread_rows<kThreads, kRows, kRows>(kt, tid, kBlk * grp, [&](int x) { return Ah + (long)src_h[min(s_base + x, S - 1)] * kD; }, q,
                                            [&] { if (tid < kRows) idx_s[tid] = src_h[min(s_base + tid, S - 1)]; });
        if (stream == 0) {
            const float inv = inv_norm(add_other_half(half_row_sumsq(q[0])));
            if (hh == 0) inv_s[kBlk * grp + l32] = inv;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i) inv_src[i] = inv_s[kBlk * grp + acc_row(i, hh)];
    };

    const int ntile = (c1 - c0 + kTileKeys - 1) / kTileKeys;
    auto multiply_tile = [&](const unsigned char *buf, int t) {
        bf16x8 kc[kSteps];
        tile_read(buf, stream, l32, hh, kc);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)   // rows = sources, columns = keys
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[0][s], kc[s], acc, 0, 0, 0);

        float sq = half_row_sumsq(kc);
        sq = add_other_half(sq);
        const float inv_k = inv_norm(sq);
        const int key = c0 + kTileKeys * t + kBlk * stream + l32;
        if (key < c1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int slot = s_base + kBlk * grp + acc_row(i, hh);
                if (slot < S) {
                    float e = (acc[i] * inv_k) * inv_src[i];
                    if (key == idx_s[kBlk * grp + acc_row(i, hh)]) e = -INFINITY;
                    E[((long)h * S + slot) * P + key] = e;
                }
            }
        }
    };
    GKV_TILE_PIPELINE(kThreads, Kh, c0, c1 - 1, 1, ntile, sources(), multiply_tile);
}

// Bound pass for ranks beyond kMaximaRank (few prompts ask for so many neighbours; others: cosine_maxima_kernel): for every
// source a value that at least m of its edges reach (short of about one
// source in 10^7, which the select catches), from the edges to a strided sample of the keys
// (column c = key c * key_stride).  `m` below is the rank in the sample that the host chose
// (mfma_bound_rank).  One workgroup takes the whole
// sample of a (head, source group): the edges never leave the registers, they are
// counted into a 256-bin histogram over [-1, 1] per source in LDS, and the bound is
// the lower edge of the bin in which the count from the top reaches m: at most 1/128
// below the m-th largest sampled edge.  (The pass is bound by the vector instructions
// that turn an edge into a bin: a plain counter per bin needs five of them per edge;
// packed 16-bit counters in twice as many bins needed eleven and made this pass 15 %
// slower for a bound that saves the filter pass 1 %.  Bins over [0, 1] only, with all
// negative edges in the lowest bin, are no option: half the updates then hit one LDS
// word.  An edge a rounding error below a bin edge may be counted into the bin above;
// the filter pass lowers every bound by far more than that.)  The source's own column
// is taken out of the counts at the end (Eq. 3: j != i).  Also clears the head's
// overflow flag for the filter pass that follows.
// One wave, one source: lane L holds the counters of bins 4L .. 4L+3 in w4 (zeros beyond the
// last bin).  Finds the bin in which the count from the top reaches m and writes its lower edge.
template <int BINS>
__device__ __forceinline__ void bound_from_histogram(const uint4 w4, int m, int lane, float *tau_row)
{
    const uint32_t c[4] = {w4.x, w4.y, w4.z, w4.w};
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mine += c[k];
    uint32_t from_top = mine;   // count in this lane's bins and all higher ones
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_down(from_top, o, kWave);
        if (lane + o < 64) from_top += v;
    }
    const uint32_t above = from_top - mine;
    if (above < (uint32_t)m && from_top >= (uint32_t)m) {
        uint32_t cum = above;
        int k = 3;
        for (; k > 0; --k) {
            if (cum + c[k] >= (uint32_t)m) break;
            cum += c[k];
        }
        *tau_row = (float)(4 * lane + k) * (2.0f / BINS) - 1.0f;
    }
    if (lane == 0 && from_top < (uint32_t)m) *tau_row = -INFINITY;   // fewer than m sampled edges: no bound
}

// Lane L's four counters of one histogram row (BINS words).
template <int BINS>
__device__ __forceinline__ uint4 histogram_words(const uint32_t *row, int lane)
{
    return lane < BINS / 4 ? *reinterpret_cast<const uint4 *>(row + 4 * lane) : make_uint4(0, 0, 0, 0);
}

// A workgroup's source rows (s_base .. of the Sh in use) against columns c0 .. c1 - 1 of the sample, counted into
// hist [ROWS][BINS].  SB 32-row groups of sources per workgroup (4 SB waves); BINS bins over [-1, 1]: 256 for two
// groups, 224 for three (the histograms of 96 rows and the two key tiles must fit the LDS), so
// the bound is at most 2 / BINS below the m-th largest sampled edge.  Ends with a barrier.
template <int SB, int BINS>
__device__ __forceinline__ void count_sample(const uint16_t *Ah, const uint16_t *Kh, const int32_t *src_h, int Sh, int s_base,
                                             int c0, int c1, int key_stride, unsigned char *kt, uint32_t *hist, float *inv_s,
                                             int32_t *idx_s, int tid)
{
    constexpr int ROWS = SB * kBlk, NT = 256 * SB;
    const int lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv & 3, grp = wv >> 2;
    bf16x8 q[kSteps];
    load_sources(Ah, src_h, Sh, s_base, grp, stream, l32, hh, q, inv_s, idx_s);
    for (int u = tid; u < ROWS * BINS; u += NT) hist[u] = 0;
    __syncthreads();
    float inv_src[16];   // 1/|k_i| times half the number of bins: edge -> bin in one multiply-add
#pragma unroll
    for (int i = 0; i < 16; ++i) inv_src[i] = inv_s[kBlk * grp + acc_row(i, hh)] * (0.5f * BINS);

    const int ntile = c1 > c0 ? (c1 - c0 + kTileKeys - 1) / kTileKeys : 0;
    auto multiply_tile = [&](const unsigned char *buf, int t) {
        bf16x8 kc[kSteps];
        tile_read(buf, stream, l32, hh, kc);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)   // rows = sources, columns = keys
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[s], kc[s], acc, 0, 0, 0);

        float sq = half_row_sumsq(kc);
        sq = add_other_half(sq);
        const float inv_k = inv_norm(sq);
        const int col = c0 + kTileKeys * t + kBlk * stream + l32;
        if (col < c1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // (e + 1) BINS / 2 with e = (dot / |k_j|) / |k_i|, the dense kernel's edge up to rounding
                int b = (int)fmaf(acc[i] * inv_k, inv_src[i], 0.5f * BINS);
                b = b < 0 ? 0 : (b > BINS - 1 ? BINS - 1 : b);
                atomicAdd(&hist[(kBlk * grp + acc_row(i, hh)) * BINS + b], 1u);
            }
        }
    };
    if (ntile > 0) GKV_TILE_PIPELINE(NT, Kh, c0, c1 - 1, key_stride, ntile, (void)0, multiply_tile);
    __syncthreads();
    // The source's own column is no neighbour (Eq. 3: j != i).  If it is one of the sampled
    // keys of this workgroup it was counted into the top bin (its edge is 1 up to rounding;
    // a zero source, all of whose edges are 0, has nothing there): take it out again.
    if (tid < ROWS) {
        const int32_t i = idx_s[tid];
        const int col = i / key_stride;
        if (i % key_stride == 0 && col >= c0 && col < c1) {
            uint32_t &top = hist[tid * BINS + BINS - 1];
            if (top > 0u) top -= 1u;
        }
    }
    __syncthreads();
}

template <int SB, int BINS>
__global__ __launch_bounds__(256 * SB) void cosine_bound_kernel(
    const uint16_t *__restrict__ Ac, const uint16_t *__restrict__ Kc, int N, int n_cols, int key_stride,
    int S, int src_pitch, const int32_t *__restrict__ src, const int32_t *__restrict__ n_src, int m,
    int chunk_cols, uint32_t *__restrict__ hist_part, float *__restrict__ tau, int pitch,
    int32_t *__restrict__ overflow)
{
    constexpr int ROWS = SB * kBlk, NT = 256 * SB;
    __shared__ float inv_s[ROWS];
    __shared__ int32_t idx_s[ROWS];
    extern __shared__ __align__(16) unsigned char smem[];   // two key tiles, then the histograms
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem + 2 * kTileBytes);   // [ROWS][BINS]

    // with few heads the sample is cut into chunks (blockIdx.z) whose histograms are added up
    // by bound_merge_kernel: otherwise a handful of workgroups would walk the sample alone
    const int h = blockIdx.y, s_base = blockIdx.x * ROWS, chunk = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c0 = chunk * chunk_cols, c1 = min(n_cols, c0 + chunk_cols);
    if (blockIdx.x == 0 && chunk == 0 && tid == 0) overflow[h] = 0;
    // rows of this head's source list in use
    const int Sh = n_src ? n_src[h] : S;
    if (s_base >= Sh) return;
    count_sample<SB, BINS>(Ac + (long)h * N * kD, Kc + (long)h * N * kD, src + (long)h * src_pitch, Sh, s_base, c0, c1,
                           key_stride, smem, hist, inv_s, idx_s, tid);

    if (gridDim.z > 1) {   // this chunk's counts go to global memory
        uint4 *out = reinterpret_cast<uint4 *>(
            hist_part + ((((long)h * gridDim.x + blockIdx.x) * gridDim.z + chunk) * ROWS) * BINS);
        const uint4 *in = reinterpret_cast<const uint4 *>(hist);
        for (int u = tid; u < ROWS * BINS / 4; u += NT) out[u] = in[u];
        return;
    }
    // Wave w scans the histograms of rows 8w .. 8w+7 from the top; lane L holds bins 4L .. 4L+3.
    for (int r = 0; r < 8; ++r) {
        const int row = wv * 8 + r;
        const uint4 w4 = histogram_words<BINS>(&hist[row * BINS], lane);
        if (s_base + row < Sh) bound_from_histogram<BINS>(w4, m, lane, &tau[(long)h * pitch + s_base + row]);
    }
}

// Adds up the histograms of the sample's chunks and takes the bound.  One
// wave per source.
template <int SB, int BINS>
__global__ __launch_bounds__(256) void bound_merge_kernel(const uint32_t *__restrict__ hist_part,
                                                          int chunks, int sgroups, int S,
                                                          const int32_t *__restrict__ n_src, int m,
                                                          float *__restrict__ tau, int pitch)
{
    constexpr int ROWS = SB * kBlk;
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * 4 + (threadIdx.x >> 6), h = blockIdx.y;
    if (slot >= (n_src ? n_src[h] : S)) return;
    const int sg = slot / ROWS, row = slot % ROWS;
    uint4 w4 = make_uint4(0, 0, 0, 0);
    for (int c0 = 0; c0 < chunks; c0 += 8) {   // (the loads of eight chunks leave together)
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = histogram_words<BINS>(
                hist_part + ((((long)h * sgroups + sg) * chunks + min(c0 + u, chunks - 1)) * ROWS + row) * BINS, lane);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (c0 + u < chunks) { w4.x += v[u].x; w4.y += v[u].y; w4.z += v[u].z; w4.w += v[u].w; }
    }
    bound_from_histogram<BINS>(w4, m, lane, &tau[(long)h * pitch + slot]);
}

// The passes below that share nothing between waves: a wave holds all source rows of its workgroup (SB groups of 32) and
// takes blocks of 32 keys of its own through a piece of LDS.
constexpr int kOwnWaves = 8;       // two per SIMD: 256 registers each
constexpr int kBlkBytes = kBlk * kPitch;

// This thread's part of the workgroup's source rows (slots beyond Sh repeat the last source).
template <int SB> struct SourcePieces {
    static constexpr int PER = SB * kBlk * 16 / (kWave * kOwnWaves);   // 16-byte pieces per thread
    u32x4 piece[PER];
    __device__ __forceinline__ void load(const uint16_t *Ah, const int32_t *src_h, int Sh, int s_base, int tid)
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int at = tid + kWave * kOwnWaves * u;
            const int32_t i = src_h[min(s_base + (at >> 4), Sh - 1)];
            piece[u] = *reinterpret_cast<const u32x4 *>(Ah + (long)i * kD + 8 * (at & 15));
        }
    }
    // Through the LDS (SB * kBlkBytes) into every wave's operand registers; 1/|k_i| of the rows to inv_s.  Read straight
    // into operand layout by every wave, 96 rows take 192 loads of 32 rows each, about 1.5 us of the start.  Ends with a barrier.
    __device__ __forceinline__ void spread(unsigned char *smem, float *inv_s, int tid, bf16x8 (&q)[SB][kSteps])
    {
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hh = lane >> 5;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int at = tid + kWave * kOwnWaves * u;
            *reinterpret_cast<u32x4 *>(smem + (at >> 4) * kPitch + (at & 15) * 16) = piece[u];
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < SB; ++g) {
            tile_read(smem, g, l32, hh, q[g]);
            if (wv == g) {
                const float inv = inv_norm(add_other_half(half_row_sumsq(q[g])));
                if (hh == 0) inv_s[kBlk * g + l32] = inv;
            }
        }
        __syncthreads();
    }
};

// Bound pass without counting: the sample is dealt out to groups of keys, 256 of them a workgroup (a group is what one
// lane position of one wave meets), every group keeps its largest edge in a register, and the bound is the rank-th
// largest of the groups' maxima -- at least `rank` sampled edges reach it, as they do the rank-th largest edge itself, and
// hardly any more do while the rank is small against the number of groups (5 % more at rank 26).  Two
// vector instructions an edge and no LDS.  (Counted into a histogram, 32 lanes hit the thirty or so bins in which the
// edges of one source lie, and the bound is only as fine as a bin.)
constexpr int kGroups = 256;
// Ranks beyond it are counted: the 64th largest of 256 maxima has 15 % more edges above it, the 62nd largest of the 128
// that parts of a sample leave 37 %.  (Counted or not, whole call of one round, us: rank 62, 128 values, 8 heads x 65504 keys
// x 64 sources 160 / 137, 64 heads 432 / 351; rank 39 of 128, 8 heads x 131008 209 / 180.)
constexpr int kMaximaRank = 64;
template <int SB> constexpr int maxima_lds_bytes() { return SB * kBlk * kGroups * 4; }   // (more than the key blocks take)

// A workgroup's source rows against n_cols >= 32 sampled keys (column c = row c * key_stride of Kh): vals [ROWS][kGroups]
// gets the groups' largest edges, -inf where a group has none.  Any 256 consecutive columns are of different
// groups, so that keys that are alike and neighbours don't hide behind one another.  Ends with a barrier.
template <int SB>
__device__ __forceinline__ void sample_maxima(const uint16_t *Ah, const uint16_t *Kh, const int32_t *src_h, int Sh, int s_base,
                                              int n_cols, int key_stride, unsigned char *smem, float *inv_s, int tid)
{
    constexpr int NW = kOwnWaves;
    static_assert(maxima_lds_bytes<SB>() >= SB * kBlkBytes, "the rows' way through the LDS");
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hh = lane >> 5;
    const int nblk = (n_cols + kBlk - 1) / kBlk;
    // (the last block of the sample starts early, as in the filter pass)
    auto block_first = [&](int b) { return min(kBlk * b, n_cols - kBlk); };
    const uint32_t row_bytes = (uint32_t)key_stride * (kD * 2), off = (uint32_t)(lane >> 4) * row_bytes + (lane & 15) * 16u;
    u32x4 stage[8];
    auto load_block = [&](int b) {
        const char *p = reinterpret_cast<const char *>(Kh) + (size_t)block_first(b) * row_bytes;
#pragma unroll
        for (int u = 0; u < 8; ++u) stage[u] = *reinterpret_cast<const u32x4 *>(p + (off + 4u * u * row_bytes));
    };
    SourcePieces<SB> sp;
    sp.load(Ah, src_h, Sh, s_base, tid);
    load_block(min(wv, nblk - 1));
    bf16x8 q[SB][kSteps];
    sp.spread(smem, inv_s, tid, q);

    float best[SB][16];
#pragma unroll
    for (int g = 0; g < SB; ++g)
#pragma unroll
        for (int i = 0; i < 16; ++i) best[g][i] = -INFINITY;
    unsigned char *mine = smem + wv * kBlkBytes;
    for (int b = wv; b < nblk; b += NW) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            *reinterpret_cast<u32x4 *>(mine + (4 * u + (lane >> 4)) * kPitch + (lane & 15) * 16) = stage[u];
        load_block(min(b + NW, nblk - 1));
        wave_sync();
        bf16x8 kc[kSteps];
        tile_read(mine, 0, l32, hh, kc);
        const int col = block_first(b) + l32;
        const float sq = add_other_half(half_row_sumsq(kc));
        const float inv_k = col >= kBlk * b ? inv_norm(sq) : NAN;   // (a maximum passes NaN by)
#pragma unroll
        for (int g = 0; g < SB; ++g) {
            f32x16 acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int s = 0; s < kSteps; ++s)   // rows = sources, columns = keys
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[g][s], kc[s], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 16; ++i) best[g][i] = fmaxf(best[g][i], acc[i] * inv_k);
        }
        wave_sync();
    }
    __syncthreads();   // the key blocks' place is free
    float *vals = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int g = 0; g < SB; ++g)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = kBlk * g + acc_row(i, hh);
            vals[row * kGroups + kBlk * wv + l32] = best[g][i] * inv_s[row];   // the dense kernel's edge
        }
    __syncthreads();
}

// Waves wv, wv + kOwnWaves, ..: the bounds of their rows < n_rows, tau_of(row, bound), from vals [n_rows][kGroups] in LDS: the
// rank-th largest value, rounded down to a multiple of 1/1024 between -1 and 1 (-inf: fewer reach -1).  Halved eleven
// times, a vote per register and step, four rows side by side so that one's votes are counted while another's compare.
// A row whose own column, which is no neighbour (Eq. 3: j != i), is among the sampled keys needs a value more.
template <typename Out>
__device__ __forceinline__ void bounds_from_maxima(const float *vals, int n_rows, const int32_t *src_rows, int key_stride, int rank,
                                                   int wv, int lane, Out &&out)
{
    constexpr int V = kGroups / kWave, RB = 4;
    for (int r0 = wv; r0 < n_rows; r0 += RB * kOwnWaves) {
        float v[RB][V];
        int need[RB], lo[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const int row = min(r0 + k * kOwnWaves, n_rows - 1);
#pragma unroll
            for (int u = 0; u < V; ++u) v[k][u] = vals[row * kGroups + lane + kWave * u];
            need[k] = rank + (src_rows[row] % key_stride == 0 ? 1 : 0);
        }
        auto reach = [&](int k, int t) {
            const float x = (float)t * (1.f / 1024.f);
            int c = 0;
#pragma unroll
            for (int u = 0; u < V; ++u) c += (int)__popcll(__ballot(v[k][u] >= x));
            return c >= need[k];
        };
        bool any[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) { lo[k] = -1024; any[k] = reach(k, -1024); }
#pragma unroll
        for (int step = 1024; step > 0; step >>= 1)
#pragma unroll
            for (int k = 0; k < RB; ++k) lo[k] = reach(k, lo[k] + step) ? lo[k] + step : lo[k];
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if (lane == 0 && r0 + k * kOwnWaves < n_rows) out(r0 + k * kOwnWaves, any[k] ? (float)lo[k] * (1.f / 1024.f) : -INFINITY);
    }
}

// The same from kParts places a row in memory, 104 to 128 of them values that the parts of a sample left: all rows of a wave
// at once through histograms of 128 bins (hist: [kOwnWaves][PER][128] words of LDS), a pair of bins a lane, then four
// halvings of the bin.  (Twelve halvings a row took 10 us of the filter pass, more than the launch that
// added up the chunks' histograms before; bounds left at the lower edge of a bin let lists of keys that are alike
// and neighbours overflow their slices.)
constexpr int kParts = 128;
template <int ROWS, typename Out>
__device__ __forceinline__ void bounds_from_parts(const float *part, int n_rows, const int32_t *src_rows, int key_stride, int rank,
                                                  uint32_t *hist, int wv, int lane, Out &&out)
{
    constexpr int PER = ROWS / kOwnWaves;
    uint2 *mine = reinterpret_cast<uint2 *>(hist + wv * PER * 128);
    float2 v[PER];
    int own[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int row = min(wv + k * kOwnWaves, n_rows - 1);
        v[k] = *reinterpret_cast<const float2 *>(part + (long)row * kParts + 2 * lane);
        own[k] = src_rows[row];
        mine[k * kWave + lane] = make_uint2(0u, 0u);
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const float x[2] = {v[k].x, v[k].y};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int b = (int)fminf((x[u] + 1.f) * 64.f, 127.f);   // (the filter pass lowers bounds by more than this rounds)
            if (x[u] >= -1.f) atomicAdd(reinterpret_cast<uint32_t *>(&mine[k * kWave]) + 127 - b, 1u);   // highest first
        }
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint2 c = mine[k * kWave + lane];
        const uint32_t need = (uint32_t)(rank + (own[k] % key_stride == 0 ? 1 : 0));
        const uint32_t upto = wave_scan_add(c.x + c.y);   // in this lane's bins and all higher ones
        const uint64_t reached = __ballot(upto >= need);
        const int row = wv + k * kOwnWaves;
        float lo = -INFINITY;
        if (reached) {   // (the same in all lanes from here on)
            const int first = __ffsll((unsigned long long)reached) - 1;
            const uint32_t high = (uint32_t)__builtin_amdgcn_readlane((int)(upto - c.y), first);
            const int bin = 127 - 2 * first - (high >= need ? 0 : 1);
            lo = (float)bin * (1.f / 64.f) - 1.f;
#pragma unroll
            for (int half = 1; half <= 4; ++half) {
                const float t = lo + 1.f / (float)(64 << half);
                if ((uint32_t)(__popcll(__ballot(v[k].x >= t)) + __popcll(__ballot(v[k].y >= t))) >= need) lo = t;
            }
        }
        if (lane == 0 && row < n_rows) out(row, lo);
    }
}

// Parts of the sample (blockIdx.z of them, every so many-th column) when there are few heads: each leaves per_chunk values
// a row in part [head, source group][ROWS][kParts], its 256 taken together by their largest, and the filter pass
// takes the bounds from all of them.  (Consecutive columns go to different parts for the same reason as to different groups.)
template <int SB>
__global__ __launch_bounds__(kWave * kOwnWaves) void cosine_maxima_kernel(
    const uint16_t *__restrict__ Ac, const uint16_t *__restrict__ Kc, int N, int n_cols, int key_stride, int S, int src_pitch,
    const int32_t *__restrict__ src, const int32_t *__restrict__ n_src, int rank, int per_chunk,
    float *__restrict__ part, float *__restrict__ tau, int pitch, int32_t *__restrict__ overflow)
{
    constexpr int ROWS = SB * kBlk, NT = kWave * kOwnWaves;
    __shared__ float inv_s[ROWS];
    extern __shared__ __align__(16) unsigned char smem[];   // key blocks, then the groups' maxima
    const float *vals = reinterpret_cast<const float *>(smem);
    const int h = blockIdx.y, s_base = blockIdx.x * ROWS, chunk = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0 && chunk == 0 && tid == 0) overflow[h] = 0;
    // rows of this head's source list in use
    const int Sh = n_src ? n_src[h] : S;
    if (s_base >= Sh) return;
    const int parts = gridDim.z;
    const int32_t *src_h = src + (long)h * src_pitch;
    sample_maxima<SB>(Ac + (long)h * N * kD, Kc + ((long)h * N + chunk * key_stride) * kD, src_h, Sh, s_base,
                      (n_cols - chunk + parts - 1) / parts, key_stride * parts, smem, inv_s, tid);
    if (parts > 1) {
        float *out = part + ((long)h * gridDim.x + blockIdx.x) * ROWS * kParts + chunk * per_chunk;
        for (int u = tid; u < ROWS * per_chunk; u += NT) {
            const int row = u / per_chunk, o = u % per_chunk;
            float best = -INFINITY;
            for (int k = o; k < kGroups; k += per_chunk) best = fmaxf(best, vals[row * kGroups + k]);
            out[row * kParts + o] = best;
        }
        if (chunk == parts - 1) {   // (and nothing in what is left)
            const int left = kParts - per_chunk * parts;
            for (int u = tid; u < ROWS * left; u += NT) out[(u / left) * kParts + per_chunk + u % left] = -INFINITY;
        }
        return;
    }
    float *tau_h = tau + (long)h * pitch + s_base;
    bounds_from_maxima(vals, min(ROWS, Sh - s_base), src_h + s_base, key_stride, rank, wv, lane, [&](int row, float t) { tau_h[row] = t; });
}

// Filter pass over all keys, barrier-free: a wave holds all source rows of its workgroup (SB groups of 32) in
// registers and takes key blocks of 32 on its own, copying each through a piece of LDS that nobody else touches.
// The loads of its next block are in flight while it works on one; the eight waves of a workgroup share nothing
// but the candidate counters, so that one wave's matrix instructions run beside another's vector work and LDS
// round trips, and the key norms are formed once per key and not once per row group.  (Tiles of 128 keys shared
// by twelve waves behind a barrier each, a wave per stream and row group: the waves loaded, multiplied, tested
// and parked in step, 1.6 us per tile of 96 rows whatever bound the call.  256 heads x 96 rows x 32736 keys 467 -> 370 us
// with the keys kept out of the caches, 362 without a hit; x 192 rows x 131008 keys 3290 -> 2430, where the matrix
// core is busy 37 % of the time at 1.7 GHz, or 53 % at the 1.46 GHz that the chip sustains without a hit, 2000.  A
// second set of accumulators, or the drain behind the next block's loads, made no difference.)
//
// A lane holds, per key block and group, the 16 dots of its key with 16 sources.  Whether one of them may reach
// its bound is tested by the matrix core too: one more instruction adds -det_i |k_j| to the dots (det_i: what
// dot / |k_j| must reach), both factors as a sum of two bf16 numbers (error below 2^-17 of the product), with the
// bounds lowered by more than that; then the largest of the 16 results, compared as integers, has no sign bit
// where there may be a hit.  That is 8 vector instructions instead of 31 per block and group.  The few lanes with
// a possible hit park their 16 dots, the key's squared norm, the key index and the group in an LDS ring.  Every
// half-wave has a ring of its own and positions are a prefix count over the hit lanes, so parking needs no atomic.
// Once a ring holds 32 rows the wave drains both, one row per lane: the test is repeated in 32-bit floats with
// the bounds from LDS, the hits' dots become exact edges (the dense kernel's formula, bit for bit), and they are
// appended to the workgroup's own slice of each source's global candidate list (one slice per key chunk, positions
// from LDS counters, so no workgroup ever waits for another).  The source's own column may be among the
// candidates: the exact select drops it.  If a slice overflows, the head's overflow flag is raised and the head is
// redone exactly, row by row.
constexpr int kStagePitch = 80;    // bytes per parked row: 16 dots, |k|^2, key, first row of the group (76, padded)
constexpr int kRing = 64;          // rows of a ring: up to 31 waiting and a group's 32
constexpr int kFilterLdsBytes = kOwnWaves * (kBlkBytes + 2 * kRing * kStagePitch);

template <int SB> struct FilterLds {
    static constexpr int ROWS = SB * kBlk;
    float inv_s[ROWS];
    __align__(16) float det_s[ROWS];
    __align__(16) uint4 test_s[2][ROWS];   // the source's operand of the test: what each half-wave holds
    int32_t row_pos[ROWS];     // entries written to each source's slice
    int32_t idle_pos[kWave];   // takes the additions of 0 of hits that are not there
};

// x as a sum of two bf16 numbers, (rounded x, rounded rest) as a pair in one register.
__device__ __forceinline__ uint32_t two_bf16(float x)
{
    const __bf16 hi = (__bf16)x;
    const bf16x2 r = {hi, (__bf16)(x - (float)hi)};
    return __builtin_bit_cast(uint32_t, r);
}

// One chunk of head h's keys against source rows s_base .. of the Sh in use; smem: kFilterLdsBytes.
// take_bounds(): called first, by all threads; tau_of(r): bound of row s_base + r.  ONCE: no other workgroup reads these keys, so they need not stay in the L2;
// the candidate lists' lines then do until they are full (256 heads of 32768 keys 468 -> 384 us, 390 without the
// lists' stores; where a second
// workgroup finds the keys there, 128 sources and 131072 keys, 2.45 -> 2.84 ms).
template <int SB, bool ONCE, typename Take, typename TauOf>
__device__ __forceinline__ void filter_chunk(const uint16_t *Ac, const uint16_t *Kc, int N, int n_cols, const int32_t *src,
                                             int chunk_cols, const FilterArgs &fa, int h, int chunk, int Sh,
                                             int s_base, FilterLds<SB> &F, unsigned char *smem, int tid, Take &&take_bounds,
                                             TauOf &&tau_of)
{
    constexpr int ROWS = SB * kBlk, NW = kOwnWaves;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hh = lane >> 5;
    const uint16_t *Kh = Kc + (long)h * N * kD;
    const int c0 = chunk * chunk_cols, c1 = min(n_cols, c0 + chunk_cols);
    const long buf_row0 = (long)h * fa.pitch + s_base;   // this workgroup's first row of the per-row buffers
    const int nblk = (c1 - c0 + kBlk - 1) / kBlk;
    const int groups = min(SB, (Sh - s_base + kBlk - 1) / kBlk);   // row groups with sources

    // Block b, whole: the last one of a head starts early where the head's rows end (N >= 32), so that every load
    // is in bounds, and the keys in front of its own are left out below.
    auto block_first = [&](int b) { return min(c0 + kBlk * b, N - kBlk); };
    u32x4 stage[8];   // 1 KiB of consecutive keys per load
    auto load_block = [&](int b) {
        const u32x4 *p = reinterpret_cast<const u32x4 *>(Kh + (long)block_first(b) * kD);
#pragma unroll
        for (int u = 0; u < 8; ++u) stage[u] = ONCE ? __builtin_nontemporal_load(p + 64 * u + lane) : p[64 * u + lane];
    };
    load_block(min(wv, nblk - 1));

    SourcePieces<SB> sp;
    sp.load(Ac + (long)h * N * kD, src + (long)h * fa.src_pitch, Sh, s_base, tid);
    take_bounds();
    if (tid < ROWS) F.row_pos[tid] = 0;
    bf16x8 q[SB][kSteps];
    sp.spread(smem, F.inv_s, tid, q);
    if (tid < ROWS) {
        const float det = dot_bound(tau_of(min(tid, Sh - 1 - s_base)), F.inv_s[tid], s_base + tid < Sh);
        F.det_s[tid] = det;
        // The matrix core's test lets through whatever the one with det does: det lowered by more than the error of
        // the two-piece product, a constant for products that underflow, everything where det is beyond all dots
        // from below; the upper limit keeps the pieces' products finite.
        const float most = 1.15292150e18f;   // 2^60
        const float low = det > most ? most : det - 2e-5f * fabsf(det);
        const bool all = !(low >= -most);
        const uint32_t pieces = all ? 0u : two_bf16(low);
        const uint32_t hi = pieces & 0xffffu, lo = pieces >> 16;
        const uint32_t extra = all ? 0x7f80u : 0x0da2u;   // +inf / 1e-30
        F.test_s[0][tid] = make_uint4(hi | (hi << 16), lo | (lo << 16), extra, 0u);
        F.test_s[1][tid] = make_uint4(0u, 0u, 0u, 0u);   // (not the same again: infinity times 0 is none)
    }
    __syncthreads();

    unsigned char *mine = smem + wv * (kBlkBytes + 2 * kRing * kStagePitch);   // this wave's block, then its two rings
    unsigned char *ring = mine + kBlkBytes + hh * (kRing * kStagePitch);
    const uint64_t half_before = (hh ? 0xffffffff00000000ull : 0x00000000ffffffffull) & ((1ull << lane) - 1ull);
    uint2 *slice0 = fa.cand + buf_row0 * fa.row_slots + (long)chunk * fa.slice_cap;
    // rows ever parked / ever drained by the lower and the upper half-wave (same in every lane)
    int tail0 = 0, tail1 = 0, head0 = 0, head1 = 0;

    // Each half-wave turns up to 32 waiting rows of its ring into list entries, one per lane.
    auto drain = [&] {
        const int n0 = min(tail0 - head0, kBlk), n1 = min(tail1 - head1, kBlk);
        wave_sync();
        if (l32 < (hh ? n1 : n0)) {
            const unsigned char *row_mem = ring + (((hh ? head1 : head0) + l32) & (kRing - 1)) * kStagePitch;
            const float4 *vals = reinterpret_cast<const float4 *>(row_mem);
            const float4 extra = vals[4];   // |k|^2, key, group
            const float inv_k = inv_norm(extra.x);   // the dense kernel's formula
            const float norm_k = norm_for_test(__builtin_amdgcn_sqrtf(extra.x));
            const uint32_t key = __float_as_uint(extra.y);
            const int row0 = (__float_as_int(extra.z) & ~(kBlk - 1)) + 4 * hh;   // row of dot 0 (a multiple of 4)
            // bit i of `hits`: dot_i reaches what its source asks for
            uint32_t misses = 0;
#pragma unroll
            for (int v = 3; v >= 0; --v) {
                const float4 dv = vals[v], tv = *reinterpret_cast<const float4 *>(&F.det_s[row0 + 8 * v]);
                const float d4[4] = {dv.x, dv.y, dv.z, dv.w}, t4[4] = {tv.x, tv.y, tv.z, tv.w};
                misses = push_misses(misses, d4, t4, norm_k);
            }
            uint32_t hits = ~misses & 0xffffu;
            // The row's first four hits without a branch, so that their LDS reads and list
            // positions are asked for together and waited for once: a hit that is not there
            // reads dot 0 and adds 0 to a counter nobody reads (one per lane).
            int rowk[4];
            int32_t atk[4];
            float dotk[4], invk[4];
            uint32_t validk = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool valid = hits != 0;
                const int i = valid ? __ffs(hits) - 1 : 0;
                hits &= hits - 1;
                validk |= valid ? 1u << k : 0u;
                rowk[k] = row0 + acc_row(i, 0);
                dotk[k] = reinterpret_cast<const float *>(row_mem)[i];
                invk[k] = F.inv_s[rowk[k]];
                atk[k] = atomicAdd(valid ? &F.row_pos[rowk[k]] : &F.idle_pos[lane], valid ? 1 : 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(dotk[k]), "+v"(invk[k]), "+v"(atk[k]));
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (((validk >> k) & 1u) && atk[k] < fa.slice_cap)
                    slice0[rowk[k] * fa.row_slots + atk[k]] =
                        make_uint2(__float_as_uint((dotk[k] * inv_k) * invk[k]), key);
            while (hits) {   // keys close to many sources at once
                const int i = __ffs(hits) - 1;
                hits &= hits - 1;
                const int row = row0 + acc_row(i, 0);
                const float e = (reinterpret_cast<const float *>(row_mem)[i] * inv_k) * F.inv_s[row];
                const int at = atomicAdd(&F.row_pos[row], 1);
                if (at < fa.slice_cap) slice0[row * fa.row_slots + at] = make_uint2(__float_as_uint(e), key);
            }
        }
        wave_sync();
        head0 += n0;
        head1 += n1;
    };

    for (int b = wv; b < nblk; b += NW) {
        // the block that has arrived -> this wave's LDS; the loads of the next one leave at once (the last block
        // again past the end), behind a drain's stores: waiting for them then waits for nothing newer
#pragma unroll
        for (int u = 0; u < 8; ++u)
            *reinterpret_cast<u32x4 *>(mine + (4 * u + (lane >> 4)) * kPitch + (lane & 15) * 16) = stage[u];
        if (tail0 - head0 >= kBlk || tail1 - head1 >= kBlk) drain();
        load_block(min(b + NW, nblk - 1));
        wave_sync();
        bf16x8 kc[kSteps];
        tile_read(mine, 0, l32, hh, kc);
        const float sq = add_other_half(half_row_sumsq(kc));
        // the key's operand of the test: -|k| in two pieces against each piece of det, 1 against the constant
        const uint32_t pieces = two_bf16(-__builtin_amdgcn_sqrtf(sq));
        u32x4 ke = {hh ? 0u : pieces, hh ? 0u : pieces, hh ? 0u : 0x3f80u, 0u};
        const int key = block_first(b) + l32;
        // (norms beyond 2^59 or NaN: left to the drain's test)
        const bool in_block = key >= c0 + kBlk * b && key < c1, sure = !(sq < 1e35f);
#pragma unroll
        for (int g = 0; g < SB; ++g) {
            if (g > 0 && g >= groups) break;
            u32x4 qe = *reinterpret_cast<const u32x4 *>(&F.test_s[hh][kBlk * g + l32]);
            f32x16 acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int s = 0; s < kSteps; ++s)   // rows = sources, columns = keys
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[g][s], kc[s], acc, 0, 0, 0);
            // dot - det |k_j| (the upper half-wave's part of the operands is 0)
            const f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, qe),
                                                                     __builtin_bit_cast(bf16x8, ke), acc, 0, 0, 0);
            int best = __float_as_int(d[0]);
#pragma unroll
            for (int i = 1; i < 16; ++i) best = max(best, __float_as_int(d[i]));
            const bool hit = (best >= 0 || sure) && in_block;
            const uint64_t hit_lanes = __ballot(hit);
            const int add0 = (int)__popcll(hit_lanes & 0x00000000ffffffffull), add1 = (int)__popcll(hit_lanes >> 32);
            // a ring that could not take these rows is drained first: one pass takes up to
            // 32 rows out, after which the (at most 32) new rows fit
            if (tail0 - head0 + add0 > kRing || tail1 - head1 + add1 > kRing) drain();
            if (hit) {
                const int at = (hh ? tail1 : tail0) + (int)__popcll(hit_lanes & half_before);
                unsigned char *row_mem = ring + (at & (kRing - 1)) * kStagePitch;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    *reinterpret_cast<float4 *>(row_mem + 16 * v) =
                        make_float4(acc[4 * v], acc[4 * v + 1], acc[4 * v + 2], acc[4 * v + 3]);
                *reinterpret_cast<float4 *>(row_mem + 64) =
                    make_float4(sq, __int_as_float(key), __int_as_float(kBlk * g), 0.f);
            }
            tail0 += add0;
            tail1 += add1;
        }
    }
    drain();
    drain();
    __syncthreads();      // every candidate is counted
    if (tid < ROWS && s_base + tid < Sh) {
        const int c = F.row_pos[tid];
        fa.cand_cnt[(buf_row0 + tid) * fa.chunk_slots + chunk] = c < fa.slice_cap ? c : fa.slice_cap;
        if (c > fa.slice_cap) fa.overflow[h] = 1;
    }
}

template <int SB, bool ONCE>
__global__ __launch_bounds__(kWave * kOwnWaves) void cosine_filter_kernel(
    const uint16_t *__restrict__ Ac, const uint16_t *__restrict__ Kc, int N, int n_cols, int S,
    const int32_t *__restrict__ src, int chunk_cols, FilterArgs fa)
{
    constexpr int ROWS = SB * kBlk;
    __shared__ FilterLds<SB> F;
    extern __shared__ __align__(16) unsigned char smem[];   // key blocks and rings, wave by wave
    // The workgroups that stream the same keys (the source groups of a key chunk) should run at
    // about the same time on the same XCD, so that all but the first find the keys in that XCD's
    // L2.  Workgroups go to the 8 XCDs round robin in the order of their linear number, so the
    // groups of one (head, chunk) unit sit 8 apart: 8 units x all their groups take 8 x sgroups
    // consecutive numbers.  (Unit counts that are no multiple of 8 keep the plain order.)
    const int n_chunks = gridDim.x / fa.sgroups;
    int h = blockIdx.y, chunk = blockIdx.x / fa.sgroups, s_base = (blockIdx.x % fa.sgroups) * ROWS;
    if (fa.sgroups > 1 && ((long)gridDim.y * n_chunks) % 8 == 0) {
        const long lin = (long)blockIdx.y * gridDim.x + blockIdx.x;
        const long grp8 = lin / (8 * fa.sgroups);
        const int r = (int)(lin % (8 * fa.sgroups));
        const long unit = grp8 * 8 + (r & 7);
        h = (int)(unit / n_chunks);
        chunk = (int)(unit % n_chunks);
        s_base = (r >> 3) * ROWS;
    }
    if (chunk * chunk_cols >= n_cols) return;
    const int Sh = fa.n_src ? fa.n_src[h] : S;
    if (s_base >= Sh) return;
    __shared__ float tau_s[ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto take_bounds = [&] {
        if (fa.part) {
            static_assert(ROWS * 128 * 4 <= kFilterLdsBytes, "the histograms take the blocks' and rings' place");
            bounds_from_parts<ROWS>(fa.part + ((long)h * fa.sgroups + s_base / ROWS) * ROWS * kParts, min(ROWS, Sh - s_base),
                                    src + (long)h * fa.src_pitch + s_base, fa.key_stride, fa.rank,
                                    reinterpret_cast<uint32_t *>(smem), wv, lane, [&](int row, float t) { tau_s[row] = t; });
            __syncthreads();
        } else if (tid < ROWS && s_base + tid < Sh) {
            tau_s[tid] = fa.tau[(long)h * fa.pitch + s_base + tid];
        }
    };
    filter_chunk<SB, ONCE>(Ac, Kc, N, n_cols, src, chunk_cols, fa, h, chunk, Sh, s_base, F, smem, tid, take_bounds,
                           [&](int r) { return tau_s[r]; });
}

// How a candidate row's entries lie: in one slice per key chunk of the pass that listed them.  From the second round on the
// rows below `late_rows` hold lists of that round's own pass.
struct Slices {
    long row_slots;
    int chunk_slots, chunks, slice_cap, late_rows, late_chunks, late_cap;
    __device__ __forceinline__ int chunks_of(int row) const { return row < late_rows ? late_chunks : chunks; }
    __device__ __forceinline__ int cap_of(int row) const { return row < late_rows ? late_cap : slice_cap; }
};

constexpr int kTieRoom = 64;   // entries tied at the cut that a select lists beyond the m winners

__device__ __forceinline__ uint32_t ord_key_u(uint32_t bits)
{
    float f = __uint_as_float(bits) + 0.0f;
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inverse of the map above (the bits of the float a key stands for).
__device__ __forceinline__ uint32_t ord_key_inv(uint32_t k)
{
    return (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
}

// Exact top-m of one source's candidate list by (edge desc, key index asc),
// written in ascending key order.  The workgroups of a head share its sources in
// turn (a workgroup's next list is asked for while it works on the current one);
// heads whose overflow flag is set are left to the exact fallback.
//
// The m-th largest edge value is found by a radix select over the order-
// preserving keys of the (short) list, as in the row top-k; entries above it are
// in, and of the entries equal to it the `need` lowest key indices are in.  The
// winners' output position is their rank by key index among themselves.
//
// The x-th selection of a head takes candidate row sel.row[h, x] of the per-row buffers
// (`pitch` rows per head) and writes the list of source slot sel.pos[h, x] of this round
// (src [Hkv, S]); without those lists row x goes to slot x.
__global__ __launch_bounds__(256) void nbr_select_kernel(const uint2 *__restrict__ cand,
                                                         const int32_t *__restrict__ cand_cnt,
                                                         int32_t *__restrict__ overflow,
                                                         const int32_t *__restrict__ src, int S, int pitch,
                                                         Slices sl, int cap, int m, SelectRows sel, int32_t *__restrict__ nbr,
                                                         float *__restrict__ nbr_e)
{
    extern __shared__ __align__(8) uint32_t dyn[];
    __shared__ uint32_t hist[256];   // 8-bit digits: the lists are short
    __shared__ uint32_t s_bin, s_need, s_min[4], s_max[4];
    __shared__ int32_t n_win;
    __shared__ int32_t end_s[256], wave_tot[4], s_pos;   // end_s[c]: entries in slices 0 .. c
    __shared__ uint32_t s_self;
    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n_rows = sel.n_rows ? sel.n_rows[h] : S;
    if (overflow[h]) return;
    // Only the edge keys of a list stay in LDS (half the footprint, twice the workgroups per
    // compute unit); the key indices of the winners, and of entries tied at the cut, are fetched
    // from the slices again once those are known.
    uint32_t *ek = dyn;                 // [cap] order-preserving edge keys (0 = dropped)
    uint64_t *win = reinterpret_cast<uint64_t *>(dyn + cap + (cap & 1));   // [m + kTieRoom] winners
    const int win_cap = m + kTieRoom;

    // candidate row and output slot of a selection, then its slice sizes (thread c: chunk c) and
    // the source's own index: two rounds of independent loads, asked for one selection ahead
    auto ask = [&](int x, int32_t &cnt_r, int32_t &self_r, int32_t &pos_r, int32_t &crow_r) {
        const long at = (long)h * S + x;
        crow_r = sel.row ? sel.row[at] : x;
        pos_r = sel.pos ? sel.pos[at] : x;
        cnt_r = tid < sl.chunks_of(crow_r) ? cand_cnt[((long)h * pitch + crow_r) * sl.chunk_slots + tid] : 0;
        self_r = src[(long)h * S + pos_r];
    };
    int32_t cnt_r = 0, self_r = 0, pos_r = 0, crow_r = 0;
    int search_steps = 0;   // bisection steps over the slices
    while ((1 << search_steps) < sl.chunk_slots) ++search_steps;
    const int wg = (int)((blockIdx.x + h) % gridDim.x);   // (few rows a head: on all XCDs)
    if (wg < n_rows) ask(wg, cnt_r, self_r, pos_r, crow_r);

    for (int x = wg; x < n_rows; x += gridDim.x) {
        const long row = (long)h * pitch + crow_r;
        const int chunks = sl.chunks_of(crow_r), slice_cap = sl.cap_of(crow_r);
        int incl = cnt_r;   // running total of the slice sizes
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += v;
        }
        if (lane == 63) wave_tot[wv] = incl;
        if (tid == 0) { s_self = (uint32_t)self_r; s_pos = pos_r; n_win = 0; }
        __syncthreads();
        for (int u = 0; u < wv; ++u) incl += wave_tot[u];
        end_s[tid] = incl;
        __syncthreads();
        if (x + (int)gridDim.x < n_rows) ask(x + gridDim.x, cnt_r, self_r, pos_r, crow_r);
        const int n = end_s[255];
        if (n > cap) {          // more candidates than the select can hold: the head is redone exactly
            if (tid == 0) overflow[h] = 1;
            return;
        }
        const uint32_t self = s_self;
        const long out_row = (long)h * S + s_pos;
        const uint2 *slices = cand + row * sl.row_slots;
        // where entry r of the concatenated slices sits: the first slice that ends behind it
        auto locate = [&](int r) {
            int lo = 0, hi = chunks - 1;
            for (int s = 0; s < search_steps; ++s) {
                const int mid = (lo + hi) >> 1;
                if (end_s[mid] > r) hi = mid; else lo = mid + 1;
            }
            lo = min(lo, chunks - 1);
            return (long)lo * slice_cap + (r - (lo ? end_s[lo - 1] : 0));
        };
        uint32_t kmin = 0xffffffffu, kmax = 0u;
        // four entries per thread and turn, their loads in flight together (entries past the
        // end read the last one again and are left out below)
        for (int r0 = tid; r0 < n; r0 += 1024) {
            uint2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = slices[locate(min(r0 + 256 * u, n - 1))];
#pragma unroll
            for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(v[u].x), "+v"(v[u].y));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = r0 + 256 * u;
                if (r < n) {
                    // the source's own column is no neighbour (Eq. 3: j != i): key 0 sorts below every edge
                    const uint32_t k = v[u].y == self ? 0u : ord_key_u(v[u].x);
                    ek[r] = k;
                    if (k) { kmin = min(kmin, k); kmax = max(kmax, k); }
                }
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, kWave));
            kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, kWave));
        }
        if (lane == 0) { s_min[wv] = kmin; s_max[wv] = kmax; }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) { kmin = min(kmin, s_min[u]); kmax = max(kmax, s_max[u]); }

        const uint32_t range = kmax - kmin;
        int remaining = (kmax >= kmin && range) ? 32 - __clz(range) : 0;
        uint32_t prefix = 0, mask = 0, need = (uint32_t)m;
        while (remaining > 0) {
            const int bits = remaining < 8 ? remaining : 8;
            const int shift = remaining - bits;
            const uint32_t dmask = (1u << bits) - 1u;
            hist[tid] = 0;
            __syncthreads();
            for (int r = tid; r < n; r += 256) {
                const uint32_t k = ek[r];
                if (k) {
                    const uint32_t rel = k - kmin;
                    if ((rel & mask) == prefix) atomicAdd(&hist[(rel >> shift) & dmask], 1u);
                }
            }
            __syncthreads();
            if (wv == 0) {   // bin where the count of larger-or-equal digits reaches `need`
                uint32_t tsum = 0;
                for (int b = 0; b < 4; ++b) tsum += hist[4 * lane + b];
                uint32_t incl = tsum;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t v = __shfl_down(incl, o, kWave);
                    if (lane + o < 64) incl += v;
                }
                const uint32_t excl = incl - tsum;
                if (excl < need && need <= incl) {
                    uint32_t cum = excl;
                    int b = 3;
                    for (; b > 0; --b) {
                        const uint32_t cb = hist[4 * lane + b];
                        if (cum + cb >= need) break;
                        cum += cb;
                    }
                    s_bin = 4 * lane + b;
                    s_need = need - cum;
                }
            }
            __syncthreads();
            prefix |= s_bin << shift;
            mask |= dmask << shift;
            need = s_need;
            remaining = shift;
        }
        const uint32_t tau = kmin + prefix;
        // Everything that reaches the threshold goes to the list as (entry number, edge bits);
        // its order is fixed by the final ranking.  More entries equal to the threshold than
        // the list has room for beyond m: the head is redone exactly.
        for (int r = tid; r < n; r += 256) {
            const uint32_t k = ek[r];
            if (k >= tau && k) {
                const int at = atomicAdd(&n_win, 1);
                if (at < win_cap) win[at] = ((uint64_t)(uint32_t)r << 32) | ord_key_inv(k);
            }
        }
        __syncthreads();
        const int listed = n_win;
        if (listed > win_cap || listed < m) {   // (fewer than m: the list was short of candidates)
            if (tid == 0) overflow[h] = 1;
            return;
        }
        // the key indices of the listed entries: (key index, edge bits) from here on
        for (int r = tid; r < listed; r += 256) {
            const uint64_t w = win[r];
            const uint32_t j = slices[locate((int)(w >> 32))].y;
            win[r] = ((uint64_t)j << 32) | (uint32_t)w;
        }
        __syncthreads();
        if (listed > m) {
            // Of the entries equal to the threshold only those with the lowest key indices stay:
            // one that `keep` or more tied entries precede is dropped (it then sorts behind all).
            const uint32_t tau_bits = ord_key_inv(tau);
            int n_tied = 0;
            for (int u = 0; u < listed; ++u) n_tied += (uint32_t)win[u] == tau_bits;
            const int keep = m - (listed - n_tied);
            uint32_t drop = 0u;   // bit i: entry tid + 256 i is dropped (written once all have compared)
            for (int r = tid, i = 0; r < listed; r += 256, ++i) {
                const uint64_t mine = win[r];
                if ((uint32_t)mine == tau_bits) {
                    int before = 0;
                    for (int u = 0; u < listed; ++u) {
                        const uint64_t w = win[u];
                        before += (uint32_t)w == tau_bits && w < mine;
                    }
                    if (before >= keep) drop |= 1u << i;
                }
            }
            __syncthreads();
            for (int r = tid, i = 0; r < listed; r += 256, ++i)
                if ((drop >> i) & 1u) win[r] = ~0ull;
            __syncthreads();
        }
        // each winner's rank by key index is its place in the output
        for (int r = tid; r < listed; r += 256) {
            const uint64_t mine = win[r];
            if (mine != ~0ull) {
                int pos = 0;
                for (int u = 0; u < listed; ++u) pos += win[u] < mine;
                nbr[out_row * m + pos] = (int32_t)(mine >> 32);
                nbr_e[out_row * m + pos] = __uint_as_float((uint32_t)mine);
            }
        }
        __syncthreads();   // the lists in LDS are free for the next row
    }
}

// The same select for short lists, one wave per source and no workgroup barrier: a lane
// keeps up to R candidates (edge key and node) in registers, so that a compute unit works on
// several times as many sources at once as with a workgroup per source -- the select is
// a chain of memory and LDS round trips, and only the number of chains in flight hides
// them.  Which slice an entry of the concatenated list belongs to comes from a mark at every
// slice's first entry and a running maximum over the lanes.  Everything that reaches the m-th
// largest key goes to a small LDS list per wave (m entries and room for 64 more that are tied at
// the cut), the tied entries with the lowest key indices are kept, and the winners are ranked by
// key index.  Lists longer than 64 R, with fewer than m entries, or with more ties at the cut than the
// list has room for, raise the head's overflow flag (the head is then redone exactly).
// (A walk over the slices for every register, key indices fetched a second time, scans through the
// LDS crossbar: 15.8 us for 512 lists in 32 slices each; this way 8.4 us.)
// (Key index and edge of a winner in one 64-bit word, ranked by comparing those: 222 us for 32768 lists of 420 entries,
// m = 128; indices in 32 bits, four a read: 180; the vote on the m-th largest ended when exactly m reach: 153.)
// Words for the key indices, and for the edges, of a wave's list: read four at a time, up to three past the end.
__host__ __device__ inline int wave_list_room(int m) { return (m + kTieRoom + 6) & ~3; }

template <int R>
__global__ __launch_bounds__(256) void nbr_select_wave_kernel(const uint2 *__restrict__ cand,
                                                              const int32_t *__restrict__ cand_cnt,
                                                              int32_t *__restrict__ overflow,
                                                              const int32_t *__restrict__ src, int S, int pitch,
                                                              Slices sl, int m, SelectRows sel,
                                                              int32_t *__restrict__ nbr,
                                                              float *__restrict__ nbr_e)
{
    static_assert(R == 16 || R == 32, "register groups of 16");
    // per wave: [64] slice starts, [64 R] marks (bytes), [list_room] key indices and edge bits of the list
    extern __shared__ __align__(16) uint32_t dyn[];
    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // (scalar: so are the row and its addresses)
    const int waves = (int)blockDim.x >> 6;
    const int n_rows = sel.n_rows ? sel.n_rows[h] : S;
    if (overflow[h]) return;
    const int list_cap = m + kTieRoom, list_room = wave_list_room(m);
    uint32_t *start_s = dyn + wv * (64 + 16 * R + 2 * list_room);
    uint8_t *mark_s = reinterpret_cast<uint8_t *>(start_s + 64);
    uint32_t *win_j = start_s + 64 + 16 * R, *win_e = win_j + list_room;

    // (with few rows a head their workgroups are the first of the head's; turned by the head they land on all XCDs)
    const int wg = (int)((blockIdx.x + h) % gridDim.x);
    for (int x = wg * waves + wv; x < n_rows; x += gridDim.x * waves) {
        const int crow = sel.row ? sel.row[(long)h * S + x] : x, pos = sel.pos ? sel.pos[(long)h * S + x] : x;
        const long row = (long)h * pitch + crow;
        const int chunks = sl.chunks_of(crow), slice_cap = sl.cap_of(crow);
        const uint2 *slices = cand + row * sl.row_slots;
        const int cnt = lane < chunks ? cand_cnt[row * sl.chunk_slots + lane] : 0;
        const uint32_t self = (uint32_t)src[(long)h * S + pos];
        const long out_row = (long)h * S + pos;
        const int incl = (int)wave_scan_add((uint32_t)cnt);   // slice sizes -> where each slice ends in the list
        const int n = __builtin_amdgcn_readlane(incl, 63);
        if (n > 64 * R || n < m) {   // too long for the lanes (or short of m): the head is redone exactly
            if (lane == 0) overflow[h] = 1;
            return;
        }
        const int n_it = (n + 63) >> 6;

        // Register it of lane L holds entry 64 it + L: first where it sits in the row's slices, then edge
        // bits (later the order-preserving key, 0 = no entry / dropped) and node.
        uint32_t E[R], J[R];
        if (chunks <= 8) {
            // few slices: the last one that starts at or before the entry, slice by slice in scalars
#pragma unroll
            for (int it = 0; it < R; ++it) J[it] = (uint32_t)(it * 64 + lane);
            for (int c = 1; c < chunks; ++c) {
                const int s_c = __builtin_amdgcn_readlane(incl - cnt, c), shift = c * slice_cap - s_c;
#pragma unroll
                for (int it = 0; it < R; ++it)
                    if ((it & ~3) < n_it) J[it] = it * 64 + lane >= s_c ? (uint32_t)(it * 64 + lane + shift) : J[it];
            }
        } else {
            // many: marks, a running maximum
            start_s[lane] = (uint32_t)(incl - cnt);
            for (int it = 0; it < n_it; ++it) mark_s[it * 64 + lane] = 0;
            wave_sync();
            if (cnt > 0) mark_s[incl - cnt] = (uint8_t)lane;
            wave_sync();
            uint32_t carry = 0;
#pragma unroll
            for (int it = 0; it < R; ++it) {
                J[it] = 0u;
                if (it < n_it) {   // (the same for all lanes)
                    const uint32_t c = wave_scan_op(max((uint32_t)mark_s[it * 64 + lane], carry), 0u,
                                                    [](uint32_t a, uint32_t b) { return max(a, b); });
                    carry = (uint32_t)__builtin_amdgcn_readlane((int)c, 63);
                    J[it] = (uint32_t)((int)c * slice_cap + it * 64 + lane - (int)start_s[c]);
                }
            }
        }
        // (entries past the end read one that is there: the loads of four registers leave together)
        const uint32_t some = (uint32_t)__builtin_amdgcn_readfirstlane((int)J[0]);
#pragma unroll
        for (int g = 0; g < R; g += 4) {
            if (g < n_it) {
                uint2 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = slices[(g + u) * 64 + lane < n ? J[g + u] : some];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    E[g + u] = v[u].x;
                    J[g + u] = v[u].y;
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) E[g + u] = 0u;
            }
        }
        uint32_t kmin = 0xffffffffu, kmax = 0u;
        int valid = n;
#pragma unroll
        for (int it = 0; it < R; ++it)
            if ((it & ~3) < n_it) {
                // the source's own column is no neighbour (Eq. 3: j != i): key 0 sorts below every edge
                const bool present = it * 64 + lane < n, own = present && J[it] == self;
                const uint32_t k = (present && !own) ? ord_key_u(E[it]) : 0u;
                valid -= (int)__popcll(__ballot(own));
                E[it] = k;
                kmin = min(kmin, k ? k : 0xffffffffu);
                kmax = max(kmax, k);
            }
        kmin = wave_min_u32(kmin);
        kmax = wave_max_u32(kmax);
        if (valid < m) {
            if (lane == 0) overflow[h] = 1;
            return;
        }

        uint32_t tau;
        if (n_it <= 2) tau = mth_largest_key<2>(E, kmin, kmax, m);
        else if (n_it <= 4) tau = mth_largest_key<4>(E, kmin, kmax, m);
        else if (n_it <= 8) tau = mth_largest_key<8>(E, kmin, kmax, m);
        else if (n_it <= 12) tau = mth_largest_key<12>(E, kmin, kmax, m);
        else if (n_it <= 16) tau = mth_largest_key<16>(E, kmin, kmax, m);
        else if (n_it <= 24) tau = mth_largest_key<(R > 24 ? 24 : R)>(E, kmin, kmax, m);
        else tau = mth_largest_key<R>(E, kmin, kmax, m);

        // everything that reaches tau -> LDS list, key index and edge bits, any order
        int listed = 0;
#pragma unroll
        for (int it = 0; it < R; ++it)
            if (it < n_it) {
                const bool in = E[it] >= tau;
                const uint64_t votes = __ballot(in);
                const int at = listed + (int)votes_below(votes);
                if (in && at < list_cap) {
                    win_j[at] = J[it];
                    win_e[at] = ord_key_inv(E[it]);
                }
                listed += (int)__popcll(votes);
            }
        if (listed > list_cap) {   // too many exactly equal edges at the cut
            if (lane == 0) overflow[h] = 1;
            return;
        }
        if (lane < 3) win_j[listed + lane] = ~0u;   // (fours are read below)
        wave_sync();
        if (listed > m) {
            // Of the entries equal to tau only those with the lowest key indices stay: one that
            // `keep` or more tied entries precede is dropped (a dropped entry sorts behind all).
            const uint32_t tau_bits = ord_key_inv(tau);
            int n_tied = 0;
            for (int u = 0; u < listed; ++u) n_tied += win_e[u] == tau_bits;
            const int keep = m - (listed - n_tied);
            // (decided for all entries first: a dropped one must still be counted by the others)
            uint32_t drop = 0;
            for (int r = lane, i = 0; r < listed; r += 64, ++i) {
                if (win_e[r] == tau_bits) {
                    const uint32_t mine = win_j[r];
                    int before = 0;
                    for (int u = 0; u < listed; ++u) before += win_e[u] == tau_bits && win_j[u] < mine;
                    if (before >= keep) drop |= 1u << i;
                }
            }
            wave_sync();
            for (int r = lane, i = 0; r < listed; r += 64, ++i)
                if ((drop >> i) & 1u) win_j[r] = ~0u;
            wave_sync();
        }
        // each winner's rank by key index is its place in the output
        for (int r = lane; r < listed; r += 64) {
            const uint32_t mine = win_j[r];
            if (mine != ~0u) {
                int at = 0;
                for (int u = 0; u < listed; u += 4) {
                    const uint4 w = *reinterpret_cast<const uint4 *>(win_j + u);
                    at += (w.x < mine) + (w.y < mine) + (w.z < mine) + (w.w < mine);
                }
                nbr[out_row * m + at] = (int32_t)mine;
                nbr_e[out_row * m + at] = __uint_as_float(win_e[r]);
            }
        }
        wave_sync();
    }
}

// Bound and filter passes in one launch; every workgroup takes the bounds of its rows from the whole sample itself.  In the
// first round where a head is one workgroup (S rows, the head's flag is cleared here): a launch, the way of the sources
// into the registers and the tail of a round of workgroups less.  In a later round (new sources only, n_src of
// them) for few heads: nearly always no head has one, and then what counts is the launches; with some, the walk over
// the sample is in front of every chunk's filter as long as each workgroup has a compute unit to itself.  COUNT: ranks
// beyond kMaximaRank (later rounds only).
template <int SB, bool ONCE, bool COUNT>
__global__ __launch_bounds__(kWave * kOwnWaves) void bound_filter_kernel(
    const uint16_t *__restrict__ Ac, const uint16_t *__restrict__ Kc, int N, int n_cols, int S,
    const int32_t *__restrict__ src, int chunk_cols, FilterArgs fa, int sample_cols)
{
    constexpr int ROWS = SB * kBlk;
    static_assert(maxima_lds_bytes<SB>() <= kFilterLdsBytes, "the groups' maxima take the blocks' and rings' place");
    __shared__ FilterLds<SB> F;
    __shared__ float tau_s[ROWS];
    extern __shared__ __align__(16) unsigned char smem[];   // key blocks, the groups' maxima, the filter pass's
    const int h = blockIdx.y, chunk = blockIdx.x / fa.sgroups, s_base = (blockIdx.x % fa.sgroups) * ROWS;
    const int Sh = fa.n_src ? fa.n_src[h] : S;
    if (s_base >= Sh) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t *src_h = src + (long)h * fa.src_pitch;
    if (!fa.n_src && tid == 0) fa.overflow[h] = 0;
    const uint16_t *Ah = Ac + (long)h * N * kD, *Kh = Kc + (long)h * N * kD;
    if constexpr (COUNT) {
        constexpr int BINS = 256;
        static_assert(256 * SB == kWave * kOwnWaves && 2 * kTileBytes + ROWS * BINS * 4 <= kFilterLdsBytes, "two tiles, the histograms");
        __shared__ int32_t idx_s[ROWS];
        uint32_t *hist = reinterpret_cast<uint32_t *>(smem + 2 * kTileBytes);
        count_sample<SB, BINS>(Ah, Kh, src_h, Sh, s_base, 0, sample_cols, fa.key_stride, smem, hist, F.inv_s, idx_s, tid);
        for (int r = wv; r < ROWS; r += kOwnWaves)
            bound_from_histogram<BINS>(histogram_words<BINS>(&hist[r * BINS], lane), fa.rank, lane, &tau_s[r]);
    } else {
        sample_maxima<SB>(Ah, Kh, src_h, Sh, s_base, sample_cols, fa.key_stride, smem, F.inv_s, tid);
        const float *vals = reinterpret_cast<const float *>(smem);
        bounds_from_maxima(vals, min(ROWS, Sh - s_base), src_h + s_base, fa.key_stride, fa.rank, wv, lane,
                           [&](int row, float t) { tau_s[row] = t; });
    }
    __syncthreads();
    // (The thread's number, read anew: what the first half forms of it need not live through it; with three groups a few
    // would spill.)
    int again = threadIdx.x;
    asm volatile("" : "+v"(again));
    filter_chunk<SB, ONCE>(Ac, Kc, N, n_cols, src, chunk_cols, fa, h, chunk, Sh, s_base, F, smem, again, [] {},
                           [&](int r) { return tau_s[r]; });
}

// Matching on its own, for source lists the few-winners selection does not take (S > 256).
__global__ __launch_bounds__(kMatchBlock) void match_sources_kernel(MatchArgs a, const int32_t *__restrict__ cur)
{
    extern __shared__ int32_t match_lds[];
    __shared__ int32_t wave_new[kMatchBlock / kWave], wave_fb[kMatchBlock / kWave];
    const bool bad = match_load(a, blockIdx.x, match_lds, threadIdx.x);
    __syncthreads();
    match_head<0>(a, blockIdx.x, bad, cur + (long)blockIdx.x * a.S, match_lds, nullptr, wave_new, wave_fb, Triples<0>{},
                  threadIdx.x);
}

// Columns per workgroup of the dense block: about 1024 workgroups in flight over all heads and source
// groups, at least 8 key blocks per wave.  (The filter pass's scratch is sized by it too.)
int chunk_cols_for(int Hkv, int sgroups, int n_cols)
{
    long ck = ((long)Hkv * sgroups * n_cols + 1023) / 1024;
    if (ck < 1024) ck = 1024;
    if (ck > n_cols) ck = n_cols;
    ck = ((ck + 127) / 128) * 128;
    return (int)(ck < 128 ? 128 : ck);
}

// Columns per workgroup of the filter pass, whole blocks for each of its waves, at most `most` chunks a head.  A compute
// unit runs one workgroup at a time, and each pays for its sources and its last drains about as long as 768 keys take:
// the cut with the fewest keys per compute unit, counting whole rounds of 256 workgroups.  (1024 workgroups of at least
// 1024 keys before; whole pass, us, before / now: 8 heads of 16K keys 106.4 / 97.5, 24 of 32K 256 / 234, 40 of 32K 382 /
// 327; at least four rounds instead: 105.7, 245, 350, and 256 heads of 20K 1013 / 999, of 32K 1399 / 1403.)
int filter_cols_for(int Hkv, int sgroups, int P, int most)
{
    const long units = (long)Hkv * sgroups, r0 = (units + 255) / 256;
    long best = -1;
    int cols = 0;
    for (long r = r0; r < r0 + 8; ++r) {
        long chunks = r * 256 / units;
        if (chunks > most) chunks = most;
        const long ck = ((P + chunks - 1) / chunks + 255) / 256 * 256;
        const long rounds = (units * ((P + ck - 1) / ck) + 255) / 256;
        const long cost = rounds * (ck + 768);
        if (best < 0 || cost < best) { best = cost; cols = (int)ck; }
    }
    return cols;
}

}  // namespace

// Most keys in the strided sample of the bound pass: every 8th key, between 2048 and 8192 keys (one
// workgroup walks the whole sample of a head's sources).  A denser sample costs the bound pass
// more and gives a tighter bound, i.e. fewer candidates for the filter pass to park and list
// (measured at 131008 keys and m = 128: 8192 sampled keys 10.2 ms per 32-layer pass, 16384 keys
// 10.4 ms, 4096 keys 10.3 ms).
int mfma_sample_cols(int P)
{
    int ps = ((P / 8 + 127) / 128) * 128;
    if (ps < 2048) ps = 2048;
    if (ps > 8192) ps = 8192;
    return ps;
}

// The sample: every stride-th key of the whole row.  (The stride rounded down would
// leave up to half of the row's end out, and a source whose near keys sit there -- neighbours in position, as
// rotary position codes make them -- gets a bound far too low: lists overflow and heads are redone row by
// row.  One round of 40 heads x 72 sources x 4064 keys in runs of 250 alike: 562 us, 181 with the whole row sampled.)
struct Sample { int stride, cols; };
static Sample sample_of(int P)
{
    const int most = mfma_sample_cols(P), stride = (P + most - 1) / most;
    return {stride, (P + stride - 1) / stride};
}

// Rank of the sampled edge that the bound is taken at.  The bound is useful for a source when at
// least m of its edges lie above it, i.e. when fewer than `rank` of its m - 1 largest edges fell
// into the sample.  With every stride-th key sampled that count is binomial, (m - 1) trials at
// 1 / stride: the rank is its mean plus six standard deviations (and one), at most m, so that
// about one source in 10^7 comes out short -- which the select notices (fewer than m candidates)
// and answers by redoing the head exactly, like an overflow.  About rank * stride keys lie above
// the rank-th sampled edge instead of m * stride: fewer rows to park, list and select from.  (Above the rank-th
// largest of V groups' maxima lie -V ln(1 - rank / V) * stride: 5 % more at rank 26 of 256, 15 % at 64, 37 % at 62 of the 128
// that parts of the sample leave, 55 % at the most, 64 of 104.)
int mfma_bound_rank(int m, int stride)
{
    if (stride <= 1) return m;
    const double mean = (m - 1.0) / stride, dev = sqrt(mean * (1.0 - 1.0 / stride));
    const int rank = (int)ceil(mean + 6.0 * dev) + 1;
    return rank < m ? rank : m;
}

int mfma_cand_cap(int P, int m)
{
    // about four times the rank * stride keys above the rank-th sampled edge (maxima of groups let up to 55 % more
    // through, bins of a histogram a few hundred at long prompts; here the stride is rounded down)
    const int stride = P / mfma_sample_cols(P);
    long cap = 4L * mfma_bound_rank(m, stride) * stride;
    if (cap < 1024) cap = 1024;
    return (int)cap;
}

// `rows`: source rows of the whole launch (heads x sources).  Short prompts (2048 <= P < 8192) take
// the filter route when their edge block would be large, from 2^23 edges (32 MiB) on: the dense
// route writes and re-reads the block, the filter route costs two more launches.  Measured (one round,
// us, dense / filter): 8 heads x 128 sources x 4064 keys (4 M edges) 117 / 119, 16 x 128 x 2968
// (6 M) 120 / 123, 32 x 64 x 4064 (8 M) 105 / 100, 64 x 64 x 2068 (8 M) 100 / 97, 64 x 64 x 7968
// (33 M) 299 / 150, 256 x 64 x 7968 (131 M) 1055 / 382.
bool mfma_filter_applies(int P, int m, long rows)
{
    // The sample must hold far more than m keys for its m-th largest edge to be a
    // useful bound, a head's rows must lie within the 32-bit byte offsets of the tile
    // loads, and the select kernel's LDS must hold a full list.
    if (P < 2048 || P >= (1 << 24)) return false;
    if (P < 8192 && rows * P < (8L << 20)) return false;
    if (m > mfma_sample_cols(P) / 8) return false;
    return (size_t)mfma_cand_cap(P, m) * 8 + (size_t)m * 8 + 8 <= 140 * 1024;
}

bool source_reuse_applies(int S) { return S <= 4096; }   // the previous list and the match's bookkeeping sit in LDS

constexpr long kManyChunksBytes = 32L << 20;

// Geometry of the filter route for a call.  X speculative rows (see the head of this file)
// ride along in the first round when the lists are kept from round to round and the extended
// source list still fits the small-k source selection; their workgroups then carry three
// 32-row groups.  Key chunks per head and the capacity of one (row, chunk) slice: four times
// the expected share of a chunk, at least 2 m (and 64) entries.
MfmaFilterPlan mfma_filter_plan(int Hkv, int P, int S, int m, bool keep_lists, bool speculate,
                                bool short_slices)
{
    MfmaFilterPlan g{};
    g.S = S;
    // speculative rows: at least one 32-row block; the extended list fills whole 96-row workgroups
    // where that takes at most two blocks
    g.X = 0;
    if (keep_lists && speculate && S + kSpecRows <= kMaxExtSources) {
        int x = (S + kSpecRows + 95) / 96 * 96 - S;
        if (x > 2 * kSpecRows) x = 2 * kSpecRows;
        if (S + x > kMaxExtSources) x = (kMaxExtSources - S) / 8 * 8;
        g.X = x;
    }
    g.sb = g.X > 0 ? 3 : 2;
    g.pitch = S + g.X;
    const int rows_wg = kBlk * g.sb;
    const int sgroups = (S + g.X + rows_wg - 1) / rows_wg;
    g.cand_cap = mfma_cand_cap(P, m);
    // a slice holds four times its expected share of a row's ~rank * stride candidates (rank: the
    // bound pass's rank in the sample), and 2 m on top
    const int stride = P / mfma_sample_cols(P);
    const long listed = (long)mfma_bound_rank(m, stride) * stride;
    auto slice_for = [&](int chunks) {
        long sc = 4L * ((listed + chunks - 1) / chunks) + 2L * m;
        if (sc < 64) sc = 64;
        // Short prompts: a row's slices may take what its row of the dense edge block would (whole 128-byte lines),
        // which holds most lists whose entries all sit in one chunk (the round above: 181 -> 94 us, in runs of 1000
        // alike 568 -> 97; keys in random order take 92 either way).
        if (P < 8192 && !short_slices && sc < P / (2 * chunks)) sc = P / (2 * chunks) / 16 * 16;
        return sc > g.cand_cap ? (long)g.cand_cap : sc;
    };
    // The memory for a row's slices is what this cut's take (at most 256 of them: the exact select keeps the slice sizes
    // of a source in LDS), and a later round's passes make no fewer chunks: a few heads with new sources among many
    // without must not be a workgroup each.  The first round's pass makes more chunks than that only where their
    // slices take little; with fewer chunks a slice is the longer.
    int cols = chunk_cols_for(Hkv, sgroups, P), chunks = (P + cols - 1) / cols;
    if (chunks > 256) {
        cols = (((P + 255) / 256 + 127) / 128) * 128;
        chunks = (P + cols - 1) / cols;
    }
    g.late_cols = g.chunk_cols = cols;
    g.late_chunks = g.chunks = g.chunk_slots = chunks;
    g.late_slice_cap = g.slice_cap = (int)slice_for(chunks);
    g.row_slots = (long)chunks * g.slice_cap;
    if (short_slices) return g;
    int most = 256;
    while (most > chunks && (long)Hkv * g.pitch * most * slice_for(most) * 8 > kManyChunksBytes) most = most / 2 > chunks ? most / 2 : chunks;
    g.chunk_cols = filter_cols_for(Hkv, sgroups, P, most);
    g.chunks = (P + g.chunk_cols - 1) / g.chunk_cols;
    if (g.chunks > chunks) {
        g.late_cols = g.chunk_cols;
        g.late_chunks = g.chunk_slots = g.chunks;
        g.late_slice_cap = g.slice_cap = (int)slice_for(g.chunks);
        g.row_slots = (long)g.chunks * g.slice_cap;
    } else {
        g.slice_cap = (int)(g.row_slots / g.chunks);
    }
    return g;
}

hipError_t launch_mfma_cosine(const void *Ac, const void *Kc, int Hkv, int N, int P, int S, const int32_t *src,
                              float *E, hipStream_t st)
{
    const int sgroups = (S + kRows - 1) / kRows;
    // One workgroup per compute unit while that leaves each a tile (a layer of a short prompt: 8 heads of
    // 4064 keys 15.4 -> 7.3 us against chunks of at least 1024 keys, which keep 32 units busy).
    int ck = chunk_cols_for(Hkv, sgroups, P);
    const long one = ((long)Hkv * sgroups * P + 255) / 256;
    if (one < 1024) ck = (int)((one + kTileKeys - 1) / kTileKeys * kTileKeys);
    const int chunks = (P + ck - 1) / ck;
    if (!allow_big_lds((const void *)cosine_dense_kernel)) return hipGetLastError();
    hipLaunchKernelGGL(cosine_dense_kernel, dim3(chunks, Hkv, sgroups), dim3(kThreads), 2 * kTileBytes,
                       st, (const uint16_t *)Ac, (const uint16_t *)Kc, N, P, S, src, ck, E);
    return hipGetLastError();
}

namespace {

// Chunks of the sample per (head, source group): 1 when the heads alone give 128 workgroups or
// more, else enough for about 256 workgroups, at least two key tiles each.
int bound_chunks(int Hkv, int P, int sgroups)
{
    const int ps = mfma_sample_cols(P);
    if (Hkv * sgroups >= 128) return 1;
    int chunks = 256 / (Hkv * sgroups);
    if (chunks > ps / (2 * kTileKeys)) chunks = ps / (2 * kTileKeys);
    return chunks < 1 ? 1 : chunks;
}

// Chunks of the sample whose maxima the filter pass puts together itself (1: the bound pass writes the bounds).  In later
// rounds there are usually no sources without a list, and one workgroup walks the whole sample.  (With a sample half as
// large more of the lists of such sources overflow: three enhanced rounds of 8 heads, mean of eight inputs, us, half /
// whole sample: 32736 keys 367 / 338, 65504 469 / 415, 131040 719 / 546, and no difference where there are none.)
int maxima_chunks(int Hkv, int P, int sgroups, int rank, bool late)
{
    return late || rank > kMaximaRank ? 1 : min(bound_chunks(Hkv, P, sgroups), kParts / 2);
}
// As many values a chunk as there is room for: 104 to 128 in all with the at most 32 chunks there are.  (Powers of two leave
// 68 of 17 chunks, and the 62nd largest of those, for 240 neighbours among 65504 keys, lets 1278 keys through on
// average and fills the longest list once in 60 rows, whose head is then redone: 15 heads with 64 sources 412 us.  119
// values let 692 through, 1022 at most in 1500 rows, and 128 672.)
int values_per_chunk(int chunks) { return kParts / chunks; }

template <int SB>
hipError_t launch_maxima(const void *Ac, const void *Kc, int Hkv, int N, int P, int rows, int rank, const int32_t *src,
                         int src_pitch, const int32_t *n_src, bool late, void *part, float *tau, int pitch, int32_t *overflow,
                         hipStream_t st)
{
    constexpr int ROWS = SB * kBlk;
    const Sample smp = sample_of(P);
    const int sgroups = (rows + ROWS - 1) / ROWS, chunks = maxima_chunks(Hkv, P, sgroups, rank, late);
    if (!allow_big_lds((const void *)cosine_maxima_kernel<SB>)) return hipGetLastError();
    hipLaunchKernelGGL(cosine_maxima_kernel<SB>, dim3(sgroups, Hkv, chunks), dim3(kWave * kOwnWaves), maxima_lds_bytes<SB>(), st,
                       (const uint16_t *)Ac, (const uint16_t *)Kc, N, smp.cols, smp.stride, rows, src_pitch, src, n_src, rank,
                       values_per_chunk(chunks), (float *)part, tau, pitch, overflow);
    return hipGetLastError();
}

template <int SB, int BINS>
hipError_t launch_bound(const void *Ac, const void *Kc, int Hkv, int N, int P, int rows, int m, const int32_t *src,
                        int src_pitch, const int32_t *n_src, bool late, void *hist_part, float *tau, int pitch,
                        int32_t *overflow, hipStream_t st)
{
    constexpr int ROWS = SB * kBlk;
    const Sample smp = sample_of(P);
    const int sgroups = (rows + ROWS - 1) / ROWS;
    const int chunks = late ? 1 : bound_chunks(Hkv, P, sgroups);
    const int chunk_cols = (((smp.cols + chunks - 1) / chunks + kTileKeys - 1) / kTileKeys) * kTileKeys;
    const int rank = mfma_bound_rank(m, smp.stride);
    if (rank <= kMaximaRank)
        return launch_maxima<SB>(Ac, Kc, Hkv, N, P, rows, rank, src, src_pitch, n_src, late, hist_part, tau, pitch, overflow, st);
    if (!allow_big_lds((const void *)cosine_bound_kernel<SB, BINS>)) return hipGetLastError();
    hipLaunchKernelGGL((cosine_bound_kernel<SB, BINS>), dim3(sgroups, Hkv, chunks), dim3(256 * SB),
                       2 * kTileBytes + ROWS * BINS * 4, st, (const uint16_t *)Ac, (const uint16_t *)Kc, N, smp.cols,
                       smp.stride, rows, src_pitch, src, n_src, rank, chunk_cols, (uint32_t *)hist_part, tau, pitch,
                       overflow);
    if (chunks > 1)
        hipLaunchKernelGGL((bound_merge_kernel<SB, BINS>), dim3((rows + 3) / 4, Hkv), dim3(256), 0, st,
                           (const uint32_t *)hist_part, chunks, sgroups, rows, n_src, rank, tau, pitch);
    return hipGetLastError();
}

template <int SB>
hipError_t launch_filter(const void *Ac, const void *Kc, int Hkv, int N, int P, int rows, int m, const int32_t *src,
                         int src_pitch, const int32_t *n_src, const MfmaFilterPlan &g, bool late, bool with_bounds,
                         const void *part, const float *tau, void *cand, int32_t *cand_cnt, int32_t *overflow, hipStream_t st)
{
    const int sgroups = (rows + SB * kBlk - 1) / (SB * kBlk);
    const Sample smp = sample_of(P);
    const int rank = mfma_bound_rank(m, smp.stride), parts = maxima_chunks(Hkv, P, sgroups, rank, late);
    FilterArgs fa{n_src, tau, parts > 1 ? (const float *)part : nullptr, rank, smp.stride, (uint2 *)cand, cand_cnt, overflow,
                  g.row_slots, g.chunk_slots, late ? g.late_slice_cap : g.slice_cap, sgroups, src_pitch, g.pitch};
    const bool once = sgroups == 1 && reads_past_caches((size_t)Hkv * N * kD * 2);
    const dim3 grid((late ? g.late_chunks : g.chunks) * sgroups, Hkv), block(kWave * kOwnWaves);
    const int cols = late ? g.late_cols : g.chunk_cols;
    if (with_bounds) {
        auto *kernel = once ? bound_filter_kernel<SB, true, false> : bound_filter_kernel<SB, false, false>;
        if constexpr (SB == kSB)   // (a later round; in the first one ranks that are counted have a bound pass)
            if (rank > kMaximaRank) kernel = once ? bound_filter_kernel<SB, true, true> : bound_filter_kernel<SB, false, true>;
        if (!allow_big_lds((const void *)kernel)) return hipGetLastError();
        hipLaunchKernelGGL(kernel, grid, block, kFilterLdsBytes, st, (const uint16_t *)Ac, (const uint16_t *)Kc, N, P, rows, src,
                           cols, fa, smp.cols);
        return hipGetLastError();
    }
    auto *kernel = once ? cosine_filter_kernel<SB, true> : cosine_filter_kernel<SB, false>;
    if (!allow_big_lds((const void *)kernel)) return hipGetLastError();
    hipLaunchKernelGGL(kernel, grid, block, kFilterLdsBytes, st, (const uint16_t *)Ac, (const uint16_t *)Kc, N, P, rows, src, cols,
                       fa);
    return hipGetLastError();
}

}  // namespace

bool mfma_filter_takes_bounds(int P, int m, const MfmaFilterPlan &g)
{
    return g.chunks == 1 && g.S + g.X <= kBlk * g.sb && mfma_bound_rank(m, sample_of(P).stride) <= kMaximaRank;
}

size_t mfma_bound_scratch_bytes(int Hkv, int P, const MfmaFilterPlan &g)
{
    // (Only the passes over a full source list cut the sample into chunks.  Sized for chunks whose edges are counted; the
    // maxima of others take less.)
    const int rows = g.S + g.X, rows_wg = kBlk * g.sb, sgroups = (rows + rows_wg - 1) / rows_wg;
    const int chunks = bound_chunks(Hkv, P, sgroups);
    return chunks > 1 ? (size_t)Hkv * sgroups * chunks * rows_wg * 256 * 4 : 0;
}

hipError_t launch_mfma_cosine_bound(const void *Ac, const void *Kc, int Hkv, int N, int P, int m,
                                    const MfmaFilterPlan &g, bool first_round, const int32_t *src,
                                    const int32_t *n_src, void *hist_part, float *tau, int32_t *overflow,
                                    hipStream_t st)
{
    if (first_round && g.sb == 3)
        return launch_bound<3, 224>(Ac, Kc, Hkv, N, P, g.S + g.X, m, src, g.S + g.X, n_src, false,
                                    hist_part, tau, g.pitch, overflow, st);
    return launch_bound<2, 256>(Ac, Kc, Hkv, N, P, g.S, m, src, g.S, n_src, !first_round, hist_part, tau, g.pitch,
                                overflow, st);
}

hipError_t launch_mfma_cosine_filter(const void *Ac, const void *Kc, int Hkv, int N, int P, int m,
                                     const MfmaFilterPlan &g, bool first_round, const int32_t *src,
                                     const int32_t *n_src, const void *hist_part, const float *tau, void *cand,
                                     int32_t *cand_cnt, int32_t *overflow, hipStream_t st)
{
    const bool with_bounds = first_round && mfma_filter_takes_bounds(P, m, g);
    if (first_round && g.sb == 3)
        return launch_filter<3>(Ac, Kc, Hkv, N, P, g.S + g.X, m, src, g.S + g.X, n_src, g, false, with_bounds, hist_part, tau,
                                cand, cand_cnt, overflow, st);
    return launch_filter<2>(Ac, Kc, Hkv, N, P, g.S, m, src, g.S, n_src, g, !first_round, with_bounds, hist_part, tau, cand,
                            cand_cnt, overflow, st);
}

hipError_t launch_match_sources(const MatchArgs &a, const int32_t *cur, int Hkv, hipStream_t st)
{
    hipLaunchKernelGGL(match_sources_kernel, dim3(Hkv), dim3(kMatchBlock), (size_t)(2 * a.S + a.X) * 4, st, a, cur);
    return hipGetLastError();
}

// A compute unit for each workgroup: with more, the walks over the sample share the units with each other.  (Three
// rounds of 8 heads, us, two launches a round / one.  No new sources: 16K keys 107.7 / 103.9, 64K keys, 512 workgroups,
// 236.7 / 233.0.  Many, from key norms: 16K keys, 64 sources, 128 workgroups 221.7 / 217.5; 128 sources, 256 277 / 274;
// 192 sources, 384 372 / 418; 64K keys, 64 sources, 512 656 / 813.  The lists selected in the same launch, by the
// workgroup that finishes last: 101.3 without new sources, but 326 and 773 with 64 and 192 and many of them new.)
bool late_filter_applies(int Hkv, const MfmaFilterPlan &g)
{
    return (long)Hkv * g.late_chunks * ((g.S + kRows - 1) / kRows) <= 256;
}

hipError_t launch_late_filter(const void *Ac, const void *Kc, int Hkv, int N, int P, int m, const MfmaFilterPlan &g,
                              const int32_t *new_src, const int32_t *n_new, void *cand, int32_t *cand_cnt,
                              int32_t *overflow, hipStream_t st)
{
    return launch_filter<kSB>(Ac, Kc, Hkv, N, P, g.S, m, new_src, g.S, n_new, g, true, true, nullptr, nullptr, cand, cand_cnt, overflow,
                              st);
}

hipError_t launch_nbr_select(const void *cand, const int32_t *cand_cnt, int32_t *overflow, const int32_t *src,
                             int Hkv, int m, const MfmaFilterPlan &g, const SelectRows *rows, int32_t *nbr,
                             float *nbr_e, hipStream_t st)
{
    const int S = g.S, cap = g.cand_cap;
    const Slices sl{g.row_slots, g.chunk_slots, g.chunks, g.slice_cap, rows ? S : 0, g.late_chunks, g.late_slice_cap};
    // Short lists in at most 64 slices: a wave per list, one to a workgroup while that spreads them over the compute units
    // (up to 2048 lists), else four.  (Few selections of a later round with many heads took the other kernel before
    // the heads' first workgroups were turned to different XCDs; 256 heads, us, workgroup / wave per list then / wave now:
    // 32K prompts 16 / 20 / 10, 20K 22 / 21 / 11, 128K 83 / 151 / 47.)
    const bool few = (long)S * Hkv <= 2048;
    if (cap <= 64 * 32 && g.chunk_slots <= 64) {
        const int waves = few ? 1 : 4;
        const SelectRows sel = rows ? *rows : SelectRows{};
        int per_head = (waves == 1 ? 2048 : 8192) / Hkv;
        per_head = per_head < 1 ? 1 : (per_head > (S + waves - 1) / waves ? (S + waves - 1) / waves : per_head);
        const bool small = cap <= 64 * 16;
        const size_t lds = (size_t)waves * (64 + 16 * (small ? 16 : 32) + 2 * wave_list_room(m)) * 4;
        auto *kernel = small ? nbr_select_wave_kernel<16> : nbr_select_wave_kernel<32>;
        hipLaunchKernelGGL(kernel, dim3(per_head, Hkv), dim3(64 * waves), lds, st, (const uint2 *)cand, cand_cnt,
                           overflow, src, S, g.pitch, sl, m, sel, nbr, nbr_e);
        return hipGetLastError();
    }
    // Longer lists: the workgroups of a head share its selections in turn: few workgroups when only some
    // sources of a round need a select (most would find nothing to do), many otherwise.
    const SelectRows sel = rows ? *rows : SelectRows{};
    int per_head = (rows ? 3072 : 16384) / Hkv;
    per_head = per_head < 1 ? 1 : (per_head > S ? S : per_head);
    const size_t lds = (size_t)(cap + (cap & 1)) * 4 + (size_t)(m + kTieRoom) * 8;
    if (!allow_big_lds((const void *)nbr_select_kernel)) return hipGetLastError();
    hipLaunchKernelGGL(nbr_select_kernel, dim3(per_head, Hkv), dim3(256), lds, st, (const uint2 *)cand,
                       cand_cnt, overflow, src, S, g.pitch, sl, cap, m, sel, nbr, nbr_e);
    return hipGetLastError();
}

}  // namespace gkv
