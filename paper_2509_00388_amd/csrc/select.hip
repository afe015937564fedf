// Exact top-k of each row of a float matrix, ties to the lowest index, output in
// ascending index order.  Used for the source nodes (Eq. 2), the neighbourhoods
// (Eq. 3) and the final budgeted selection.
//
// One workgroup per row.  The sources and the edges of a dense row (few winners) come from a short list
// of the entries that reach a bound, the budgeted selection from one histogram sweep and a bitmap (see
// there).  What those do not take -- more than 256 winners with values, rows beyond 2^18 entries, masses of
// equal values, the scratch rows of the exact fallback -- goes through a most-significant-digit-first
// radix select over an order-preserving 32-bit key, whose last sweep emits, in index order, every entry
// above the threshold and the first `need` entries equal to it: exactly "first k by (value desc, index
// asc)".  All counting is integer, so no result depends on scheduling.
#include "common.hpp"
#include "decay.hpp"
#include "kernels.hpp"
#include "match.hpp"
#include "mfma_tile.hpp"

#include <type_traits>

namespace gkv {

namespace {

constexpr int kBins = 2048;   // bins of the streaming variant (11-bit digits)

// The thread's number, read anew: what is computed from it stays where it is used.  (Where a kernel begins with the
// loads of a whole row, or loops over rows, the compiler otherwise moves the addresses of much that comes later in front
// of them.  Redone rows: 146 registers a lane spill, 294 -> 334 us for 8 heads of 32736 keys; a selection that takes
// the update along: 16352 entries 25.4 -> 27.9 us with 68 registers instead of 57.)
__device__ __forceinline__ int here(int tid)
{
    asm volatile("" : "+v"(tid));
    return tid;
}

__device__ __forceinline__ float key_to_float(uint32_t key)   // inverse of ord_key
{
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// Key of an entry of a row, where 0 stands for no entry: the one value whose key is 0 (a NaN of all ones)
// gets 1, so that a row always holds as many keys as entries.
__device__ __forceinline__ uint32_t entry_key(float v) { return max(ord_key(v), 1u); }

// Histogram one digit of the keys that still match the prefix.  `in` says
// whether this lane's key takes part.  A wave whose keys all share the digit
// (usual in the top digit) issues a single add.
__device__ __forceinline__ void hist_add(uint32_t *hist, bool in, uint32_t dig, int lane)
{
    const uint64_t act = __ballot(in);
    if (!act) return;
    const int first = __ffsll((long long)act) - 1;
    const uint32_t d0 = __shfl(dig, first, kWave);
    const uint64_t same = __ballot(in && dig == d0);
    if (same == act) {
        if (lane == first) atomicAdd(&hist[d0], (uint32_t)__popcll(act));
    } else if (in) {
        atomicAdd(&hist[dig], 1u);
    }
}

// Wave 0: find the bin where the count of larger-or-equal digits reaches `need`.
// Lane L owns bins BPL*L .. BPL*L+BPL-1 (64*BPL bins in all).  Writes
// {bin, need - (entries in higher bins)}.
template <int BPL>
__device__ __forceinline__ void find_bin(const uint32_t *hist, uint32_t need, int lane,
                                         uint32_t *s_bin, uint32_t *s_need)
{
    uint32_t t = 0;
#pragma unroll
    for (int b = 0; b < BPL; ++b) t += hist[BPL * lane + b];
    uint32_t incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_down(incl, o, kWave);
        if (lane + o < 64) incl += v;
    }
    const uint32_t excl = incl - t;   // entries in strictly higher lanes
    if (excl < need && need <= incl) {
        uint32_t cum = excl;
        int b = BPL - 1;
        for (; b > 0; --b) {
            const uint32_t c = hist[BPL * lane + b];
            if (cum + c >= need) break;
            cum += c;
        }
        *s_bin = BPL * lane + b;
        *s_need = need - cum;
    }
}

}  // namespace

// ---- rows kept in LDS ---------------------------------------------------------
// The row is read once, coalesced, and its keys stay in LDS (up to 32768 entries
// = 128 KiB) for all sweeps.  Thread t handles entries i*BLOCK + t; index order is
// therefore (i, wave, lane), and the emit sweep counts per (i, wave) cell with
// ballots and scans the cells once.
// DIG = bits per radix sweep (11 for long rows, 8 for short ones: fewer bins to clear
// and scan).
template <int BLOCK, int DIG>
__device__ __forceinline__ void topk_row_lds(
    int row, const float *__restrict__ x, long ld, int n, int k, int32_t *__restrict__ idx_out,
    long idx_ld, float *__restrict__ val_out, long val_ld)
{
    constexpr int NW = BLOCK / kWave;
    constexpr int NBINS = 1 << DIG;
    extern __shared__ uint32_t dyn[];
    __shared__ uint32_t hist[NBINS];
    __shared__ uint32_t s_bin, s_need;

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int items = (n + BLOCK - 1) / BLOCK;
    const int ncell = items * NW;
    uint32_t *keys = dyn;                    // [items * BLOCK]
    uint32_t *cg = dyn + items * BLOCK;      // [ncell]
    uint32_t *ce = cg + ncell;               // [ncell]
    const float *xr = x + (long)row * ld;
    int32_t *out = idx_out + (long)row * idx_ld;
    float *vout = val_out ? val_out + (long)row * val_ld : nullptr;

    // Keys to LDS; the row's key range [kmin, kmax] on the way.
    __shared__ uint32_t s_min[NW], s_max[NW];
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll 8
    for (int i = 0; i < items; ++i) {
        const int j = i * BLOCK + tid;
        const float v = xr[min(j, n - 1)];   // (unconditional: the loads of a batch leave together)
        const uint32_t key = ord_key(j < n ? v : 0.f);
        keys[j] = key;
        if (j < n) { kmin = min(kmin, key); kmax = max(kmax, key); }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, kWave));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, kWave));
    }
    if (lane == 0) { s_min[wv] = kmin; s_max[wv] = kmax; }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NW; ++u) { kmin = min(kmin, s_min[u]); kmax = max(kmax, s_max[u]); }

    // Radix select on (key - kmin): only the bits in which the row's keys differ
    // are swept, and the top digit is spread over the bins whatever the value range.
    const uint32_t range = kmax - kmin;
    int remaining = range ? 32 - __clz(range) : 0;
    uint32_t prefix = 0, mask = 0, need = (uint32_t)k;
    while (remaining > 0) {
        const int bits = remaining < DIG ? remaining : DIG;
        const int shift = remaining - bits;
        const uint32_t dmask = (1u << bits) - 1u;
        for (int b = tid; b < NBINS; b += BLOCK) hist[b] = 0;
        __syncthreads();
        for (int i = 0; i < items; ++i) {
            const int j = i * BLOCK + tid;
            const uint32_t rel = keys[j] - kmin;
            if (j < n && (rel & mask) == prefix) atomicAdd(&hist[(rel >> shift) & dmask], 1u);
        }
        __syncthreads();
        if (wv == 0) find_bin<NBINS / 64>(hist, need, lane, &s_bin, &s_need);
        __syncthreads();
        prefix |= s_bin << shift;
        mask |= dmask << shift;
        need = s_need;
        remaining = shift;
    }
    const uint32_t tau = kmin + prefix;   // key of the k-th largest entry; take `need` entries equal to it

    for (int i = 0; i < items; ++i) {
        const int j = i * BLOCK + tid;
        const uint32_t key = keys[j];
        const uint32_t ng = __popcll(__ballot(j < n && key > tau));
        const uint32_t ne = __popcll(__ballot(j < n && key == tau));
        if (lane == 0) { cg[i * NW + wv] = ng; ce[i * NW + wv] = ne; }
    }
    __syncthreads();
    if (wv == 0) {   // exclusive scan of the cells in index order; lane L owns a contiguous run
        const int per = (ncell + 63) / 64;
        const int c0 = min(lane * per, ncell), c1 = min(c0 + per, ncell);
        uint32_t sg = 0, se = 0;
        for (int c = c0; c < c1; ++c) { sg += cg[c]; se += ce[c]; }
        uint32_t ig = sg, ie = se;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t a = __shfl_up(ig, o, kWave), b = __shfl_up(ie, o, kWave);
            if (lane >= o) { ig += a; ie += b; }
        }
        uint32_t bg = ig - sg, be = ie - se;
        for (int c = c0; c < c1; ++c) {
            const uint32_t tg = cg[c], te = ce[c];
            cg[c] = bg; ce[c] = be;
            bg += tg; be += te;
        }
    }
    __syncthreads();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    for (int i = 0; i < items; ++i) {
        const int j = i * BLOCK + tid;
        const uint32_t key = keys[j];
        const bool g = j < n && key > tau, e = j < n && key == tau;
        const uint64_t mg = __ballot(g), me = __ballot(e);
        if (g || e) {
            const uint32_t g_before = cg[i * NW + wv] + __popcll(mg & lt_mask);
            const uint32_t e_before = ce[i * NW + wv] + __popcll(me & lt_mask);
            if (g || e_before < need) {
                const uint32_t pos = g_before + min(e_before, need);
                out[pos] = j;
                if (vout) vout[pos] = key_to_float(key);
            }
        }
    }
}

// One workgroup per row.
template <int BLOCK, int DIG>
__global__ __launch_bounds__(BLOCK) void topk_rows_lds_kernel(
    const float *__restrict__ x, long ld, int n, int k, int32_t *__restrict__ idx_out, long idx_ld,
    float *__restrict__ val_out, long val_ld)
{
    topk_row_lds<BLOCK, DIG>(blockIdx.x, x, ld, n, k, idx_out, idx_ld, val_out, val_ld);
}

// ---- rows of any length: every sweep re-reads the row ------------------------
// PLAN: k and the output row come from the per-layer budgets, `append_count` consecutive integers from append_from
// on follow the k entries.
template <int BLOCK, bool PLAN>
__device__ __forceinline__ void topk_stream_row(
    int row, const float *__restrict__ x, long ld, int n, int k, int32_t *__restrict__ idx_out, long idx_ld,
    float *__restrict__ val_out, long val_ld, int append_from, int append_count,
    typename std::conditional<PLAN, LayerPlan, int>::type plan)
{
    constexpr int NW = BLOCK / kWave;
    constexpr int U = 8;   // loads in flight per thread
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t s_bin, s_need;
    __shared__ uint32_t w_gt[NW], w_eq[NW];

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float *xr = x + (long)row * ld;
    int32_t *out = idx_out + (long)row * idx_ld;
    float *vout = val_out ? val_out + (long)row * val_ld : nullptr;
    if constexpr (PLAN) {   // per-layer budget: k and the output row come from the plan
        const int g = row / plan.heads_per_layer, hl = row % plan.heads_per_layer;
        k = plan.budget[g] - append_count;
        out = idx_out + (plan.row_off[g] + (long)hl * plan.budget[g]);
        for (int r = tid; r < append_count; r += BLOCK) out[k + r] = append_from + r;
    }

    uint32_t prefix = 0, mask = 0, need = (uint32_t)k;
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
        const uint32_t dmask = pass == 2 ? 1023u : 2047u;
        for (int b = tid; b < kBins; b += BLOCK) hist[b] = 0;
        __syncthreads();
        for (int j0 = 0; j0 < n; j0 += BLOCK * U) {
            float t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u * BLOCK + tid;
                t[u] = xr[min(j, n - 1)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t key = ord_key(t[u]);
                const bool in = (j0 + u * BLOCK + tid < n) && ((key & mask) == prefix);
                hist_add(hist, in, (key >> shift) & dmask, lane);
            }
        }
        __syncthreads();
        if (wv == 0) find_bin<32>(hist, need, lane, &s_bin, &s_need);
        __syncthreads();
        prefix |= s_bin << shift;
        mask |= dmask << shift;
        need = s_need;
    }
    const uint32_t tau = prefix;

    // Each wave owns a contiguous, 64-aligned segment of the row.
    int seg = (n + NW - 1) / NW;
    seg = (seg + 63) & ~63;
    const int beg = wv * seg;
    const int end = min(n, beg + seg);

    uint32_t cgt = 0, ceq = 0;
    for (int j0 = beg; j0 < end; j0 += kWave * U) {
        float t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
            t[u] = xr[min(j, n - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
            const uint32_t key = ord_key(t[u]);
            cgt += __popcll(__ballot(j < end && key > tau));
            ceq += __popcll(__ballot(j < end && key == tau));
        }
    }
    if (lane == 0) { w_gt[wv] = cgt; w_eq[wv] = ceq; }
    __syncthreads();
    uint32_t base_g = 0, base_e = 0;
    for (int i = 0; i < wv; ++i) { base_g += w_gt[i]; base_e += w_eq[i]; }

    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int j0 = beg; j0 < end; j0 += kWave * U) {
        float t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
            t[u] = xr[min(j, n - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
            const bool live = j < end;
            const uint32_t key = ord_key(t[u]);
            const bool g = live && key > tau, e = live && key == tau;
            const uint64_t mg = __ballot(g), me = __ballot(e);
            const uint32_t g_before = base_g + __popcll(mg & lt_mask);
            const uint32_t e_before = base_e + __popcll(me & lt_mask);
            if (g || (e && e_before < need)) {
                const uint32_t pos = g_before + min(e_before, need);
                out[pos] = j;
                if (vout) vout[pos] = t[u] + 0.0f;   // (no -0.0, as everywhere else)
            }
            base_g += __popcll(mg);
            base_e += __popcll(me);
        }
    }
}

template <int BLOCK, bool PLAN>
__global__ __launch_bounds__(BLOCK) void topk_rows_stream_kernel(
    const float *__restrict__ x, long ld, int n, int k, int32_t *__restrict__ idx_out, long idx_ld,
    float *__restrict__ val_out, long val_ld, int append_from, int append_count,
    typename std::conditional<PLAN, LayerPlan, int>::type plan)
{
    topk_stream_row<BLOCK, PLAN>(blockIdx.x, x, ld, n, k, idx_out, idx_ld, val_out, val_ld, append_from, append_count,
                                 plan);
}

// A row in batches of U loads per thread of a 1024-thread workgroup, the next batch on its way
// while one is used; use(number of the 64 entries, value, in the row) is called by whole waves.  The
// batches that fill the workgroup are loaded without a condition (past the last one, the last again):
// behind a conditional load the compiler waits for everything in flight.  The few turns behind them hold
// the row's end.
template <int U, typename Use>
__device__ __forceinline__ void row_sweep(const float *__restrict__ xr, int n, int tid, int wv, Use &&use)
{
    constexpr int BLOCK = 1024, NW = BLOCK / kWave;
    const int turns = (n + BLOCK - 1) / BLOCK, whole = n / BLOCK / U * U;
    float tail[U];
#pragma unroll
    for (int u = 0; u < U; ++u) tail[u] = xr[min((whole + u) * BLOCK + tid, n - 1)];
    if (whole > 0) {
        float a[U], b[U];
        auto load = [&](float (&v)[U], int i0) {
            const float *p = xr + (long)min(i0, whole - U) * BLOCK;
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p[u * BLOCK + tid];
            __builtin_amdgcn_sched_barrier(0);
        };
        auto work = [&](float (&v)[U], int i0) {
#pragma unroll
            for (int u = 0; u < U; ++u) use((i0 + u) * NW + wv, v[u], true);
        };
        load(a, 0);
        for (int i0 = 0; i0 < whole; i0 += 2 * U) {
            load(b, i0 + U);
            work(a, i0);
            load(a, i0 + 2 * U);
            if (i0 + U < whole) work(b, i0 + U);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (whole + u < turns) use((whole + u) * NW + wv, tail[u], (whole + u) * BLOCK + tid < n);
}

// ---- few winners (source nodes) -------------------------------------------------------
// The k <= kSmallK best entries of a row, split into the S best and the X = k - S next best, each
// group in ascending index order (Eq. 2).  One workgroup of 16 waves per row.  A lower bound of the
// k-th largest key comes almost for free: every thread takes the largest key it owns, one
// histogram of those 1024 maxima finds the bin of the k-th largest of them, and at least k entries
// reach its lower edge.  The entries that do (k and a few dozen more) go to a list of (key, index)
// pairs; every thread ranks one of them against all others, which gives both the winners and their
// split, and counts the winners of lower index for its place.  What bounds it is the chain of memory
// and LDS round trips.  Rows of up to 32768 entries are read once into registers, longer ones
// twice.  (A group bound through LDS maxima, a radix sweep and one wave that finished the row
// alone, bit by bit: 21.4 us with k = 96 and 16.4 us with k = 64 for 8 rows of 32736 entries;
// this way 9.8 and 8.2 us, 7.7 and 6.2 since floats are compared and several threads share
// an entry's rank; 256 rows of 131008 entries with k = 192: 72 us before, 49 us now.)
//
// The same code takes the m best edges of a source from its row of the dense edge block (Eq. 3): 256
// threads per row of up to 8192 edges, no split, the edges' values beside their indices.  (Three LDS
// histogram sweeps per row: 14.0 us for 256 rows of 4064 edges with m = 8 and 22.5 us for 512 rows of
// 8160 with m = 16; this way 5.9 and 7.5 us.)
constexpr int kSmallK = 256;       // largest k
constexpr int kPickBlock = 1024;
constexpr int kPickList = 1024;    // entries the list takes

template <int BLOCK> struct PickLds {
    static constexpr int NW = BLOCK / kWave, kBits = BLOCK == 1024 ? 11 : 9;
    static_assert((1 << kBits) == 2 * BLOCK, "two bins per thread");
    __align__(16) uint32_t hist[2 * BLOCK];
    __align__(16) uint64_t list[kPickList];   // (key << 32) | ~index: larger = first
    __align__(16) uint32_t win[kSmallK];      // indices of the winners by rank
    uint32_t val[kSmallK];                    // their keys (edges)
    uint32_t part[2][NW], lo[NW], hi[NW], out[3], cnt;

    __device__ __forceinline__ void clear(int tid)
    {
        hist[tid] = 0;
        hist[tid + BLOCK] = 0;
#pragma unroll
        for (int u = 0; u < kPickList; u += BLOCK) list[u + tid] = 0;
        if (tid == 0) cnt = 0;
    }
};

// Where a row's winners go: sources (src, and ext unless null: the S best, then all k), or edges (nbr
// and their values).
struct PickOut {
    int S;
    int32_t *src, *ext;
    float *val;
};

// Lower edge of the bin (of 2 BLOCK over their range) that holds the k-th largest of the threads'
// values; a thread without a value passes 0.  `hist` is zero on entry.  Contains barriers.
template <int BLOCK>
__device__ __forceinline__ uint32_t kth_value_bound(uint32_t best, int k, PickLds<BLOCK> &L, int tid, int lane, int wv)
{
    constexpr int NW = PickLds<BLOCK>::NW, BITS = PickLds<BLOCK>::kBits;
    const uint32_t mn = wave_min_u32(best ? best : 0xffffffffu), mx = wave_max_u32(best);
    if (lane == 0) { L.lo[wv] = mn; L.hi[wv] = mx; }
    __syncthreads();
    const uint32_t kmin = wave_min_u32(L.lo[lane & (NW - 1)]), kmax = wave_max_u32(L.hi[lane & (NW - 1)]);
    const int bits = kmax > kmin ? 32 - __clz(kmax - kmin) : 0, shift = bits > BITS ? bits - BITS : 0;
    if (best) atomicAdd(&L.hist[(best - kmin) >> shift], 1u);
    __syncthreads();
    find_bin_block<BLOCK>(L.hist, (uint32_t)k, L.part[0], L.out, tid, lane, wv);
    return kmin + (L.out[0] << shift);
}

// Sum over groups of 2^LOG neighbouring lanes (LOG <= 3), in every lane of the group.
template <int LOG> __device__ __forceinline__ int lane_group_sum(int v)
{
#define GKV_DPP(ctrl) __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, false)
    if constexpr (LOG > 0) v += GKV_DPP(0xb1);    // quad_perm: the neighbour
    if constexpr (LOG > 1) v += GKV_DPP(0x4e);    // quad_perm: the other pair
    if constexpr (LOG > 2) v += GKV_DPP(0x141);   // row_half_mirror: the other four
#undef GKV_DPP
    return v;
}

// Ranks of the cnt listed entries -> win (and val): 2^LOG neighbouring threads share an entry.
template <int BLOCK, int LOG, bool EDGES>
__device__ __forceinline__ void rank_winners(PickLds<BLOCK> &L, int cnt, int k, int tid)
{
    constexpr int G = 1 << LOG;
    for (int t0 = 0; t0 < cnt; t0 += BLOCK / G) {   // (once if the entries fit)
        const int t = t0 + tid / G;
        const uint64_t mine = L.list[min(t, kPickList - 1)];
        int rank = 0;
        for (int u = 2 * (tid % G); u < cnt; u += 2 * G) {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(L.list + u);
            rank += (v.x > mine) + (v.y > mine);
        }
        rank = lane_group_sum<LOG>(rank);
        if (tid % G == 0 && t < cnt && rank < k) {
            L.win[rank] = ~(uint32_t)mine;
            if (EDGES) L.val[rank] = (uint32_t)(mine >> 32);
        }
    }
    __syncthreads();
}

// The k winners -> the row's outputs, by index within their group (the S best, the others).
template <int BLOCK, int LOG, bool EDGES>
__device__ __forceinline__ void place_winners(PickLds<BLOCK> &L, int k, const PickOut &o, int tid)
{
    constexpr int G = 1 << LOG;
    for (int t0 = 0; t0 < k; t0 += BLOCK / G) {
        const int t = min(t0 + tid / G, k - 1), from = EDGES || t < o.S ? 0 : o.S, to = EDGES || t >= o.S ? k : o.S;
        const uint32_t mine = L.win[t];
        int at = 0;
        for (int u = from + tid % G; u < to; u += G) at += L.win[u] < mine;
        at = from + lane_group_sum<LOG>(at);
        if (tid % G == 0 && t0 + tid / G < k) {
            if (EDGES) {
                o.src[at] = (int32_t)mine;
                o.val[at] = key_to_float(L.val[t]);
            } else {
                if (at < o.S) o.src[at] = (int32_t)mine;
                if (o.ext) o.ext[at] = (int32_t)mine;
            }
        }
    }
}

// The list of cnt >= k entries (zeros behind them) -> the row's outputs.
template <int BLOCK, bool EDGES>
__device__ __forceinline__ void emit_winners(PickLds<BLOCK> &L, int cnt, int k, const PickOut &o, int tid)
{
    if (cnt <= BLOCK / 8) rank_winners<BLOCK, 3, EDGES>(L, cnt, k, tid);
    else if (cnt <= BLOCK / 2) rank_winners<BLOCK, 1, EDGES>(L, cnt, k, tid);
    else rank_winners<BLOCK, 0, EDGES>(L, cnt, k, tid);
    if (k <= BLOCK / 8) place_winners<BLOCK, 3, EDGES>(L, k, o, tid);
    else place_winners<BLOCK, 2, EDGES>(L, k, o, tid);
}

// More entries reach the bound than the list holds, or fewer than k: a histogram over all of them raises the bound,
// or, for masses of equal values, the general algorithm picks the k entries.  Returns the entries of the list, or 0
// if the outputs are written.  The row is read again.
template <int BLOCK, bool EDGES>
__device__ __forceinline__ int pick_hard(const float *xr, int n, int k, const PickOut &o, PickLds<BLOCK> &L, uint32_t bound,
                                         int cnt)
{
    constexpr int NW = PickLds<BLOCK>::NW, BITS = PickLds<BLOCK>::kBits;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (cnt > kPickList) {
        uint32_t mx = 0u;
        for (int j = tid; j < n; j += BLOCK) mx = max(mx, ord_key(xr[j]));
        mx = wave_max_u32(mx);
        __syncthreads();
        L.clear(tid);
        if (lane == 0) L.hi[wv] = mx;
        __syncthreads();
        mx = wave_max_u32(L.hi[lane & (NW - 1)]);
        const int bits = mx > bound ? 32 - __clz(mx - bound) : 0, shift = bits > BITS ? bits - BITS : 0;
        for (int j = tid; j < n; j += BLOCK) {
            const uint32_t key = ord_key(xr[j]);
            if (key >= bound) atomicAdd(&L.hist[(key - bound) >> shift], 1u);
        }
        __syncthreads();
        find_bin_block<BLOCK>(L.hist, (uint32_t)k, L.part[0], L.out, tid, lane, wv);
        bound += L.out[0] << shift;
        for (int j = tid; j < n; j += BLOCK) {
            const uint32_t key = ord_key(xr[j]);
            if (key >= bound) {
                const uint32_t at = atomicAdd(&L.cnt, 1u);
                if (at < (uint32_t)kPickList) L.list[at] = ((uint64_t)key << 32) | (uint32_t)~j;
            }
        }
        __syncthreads();
        if (L.cnt <= (uint32_t)kPickList) return (int)L.cnt;
    }
    int32_t *tmp = !EDGES && o.ext ? o.ext : o.src;
    topk_stream_row<BLOCK, false>(0, xr, n, n, k, tmp, 0, EDGES ? o.val : nullptr, 0, 0, 0, 0);
    if (EDGES) return 0;
    __syncthreads();
    const int32_t j = tid < k ? tmp[tid] : 0;
    L.list[tid] = tid < k ? ((uint64_t)ord_key(xr[j]) << 32) | (uint32_t)~j : 0ull;   // (k <= 256 <= BLOCK)
    __syncthreads();
    return k;
}

// A row of at most ITEMS * BLOCK entries (and, with ITEMS > 2, more than half as many), entry i of thread tid being
// number i * BLOCK + tid: all its loads leave together, unconditional and clamped.
template <int BLOCK, int ITEMS>
__device__ __forceinline__ void load_row(const float *xr, int n, int tid, float (&val)[ITEMS])
{
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) val[i] = xr[min(i * BLOCK + tid, n - 1)];
}

// Its k best, from the registers; L is cleared.  Floats are compared, an instruction per entry where keys take half
// a dozen (an instruction for every entry of a row of 32768 takes a compute unit 0.2 us).  They order as their keys
// do but for NaN, which every comparison leaves out: so the maxima are those of the numbers, which can only lower
// the bound; what is not below the bound is looked at by its key, and a row in which fewer than k entries reach it
// goes through the general algorithm, by keys throughout.
template <int BLOCK, int ITEMS, bool EDGES, bool ANY = false>   // ANY: a row of any length up to ITEMS * BLOCK
__device__ __forceinline__ void pick_row(float (&val)[ITEMS], const float *xr, int n, int k, const PickOut &o,
                                         PickLds<BLOCK> &L, int tid, int lane, int wv)
{
    static_assert(ITEMS <= 32, "one bit per entry of a thread");
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) asm volatile("" : "+v"(val[i]));   // (the batch of loads stays one)
#pragma unroll
    for (int i = ITEMS > 2 && !ANY ? ITEMS / 2 : 0; i < ITEMS; ++i) val[i] = i * BLOCK + tid < n ? val[i] : -INFINITY;
    float best = -INFINITY;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) best = val[i] > best ? val[i] : best;   // (never NaN)
    const uint32_t bound_key = kth_value_bound<BLOCK>(tid < n ? ord_key(best) : 0u, k, L, tid, lane, wv);
    const float bound = key_to_float(bound_key);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (!(val[i] < bound)) {
            const uint32_t key = ord_key(val[i]);
            if (key >= bound_key && i * BLOCK + tid < n) {
                const uint32_t at = atomicAdd(&L.cnt, 1u);
                if (at < (uint32_t)kPickList) L.list[at] = ((uint64_t)key << 32) | (uint32_t)~(i * BLOCK + tid);
            }
        }
    __syncthreads();
    int cnt = (int)L.cnt;   // (the same for every thread, like all branches here)
    if (cnt < k || cnt > kPickList) {
        cnt = pick_hard<BLOCK, EDGES>(xr, n, k, o, L, bound_key, cnt);
        if (cnt == 0) return;
    }
    emit_winners<BLOCK, EDGES>(L, cnt, k, o, tid);
}

// A longer row: read twice, in batches of 12 loads per thread.  Both reads compare floats, an instruction
// less per entry than keys; floats order as their keys do but for NaN, which every comparison leaves out.
// So the maxima are those of the numbers, which can only lower the bound; what is not below the bound is
// looked at by its key, and a row in which fewer than k entries reach it goes through the general algorithm,
// by keys throughout.
__device__ __forceinline__ void pick_row_long(const float *xr, int n, int k, const PickOut &o, PickLds<kPickBlock> &L,
                                              int tid, int lane, int wv)
{
    L.clear(tid);
    float best = -INFINITY;
    row_sweep<12>(xr, n, tid, wv, [&](int, float v, bool in) { best = fmaxf(best, in ? v : -INFINITY); });
    // (the bound need not be the key of an entry)
    const uint32_t bound_key = kth_value_bound<kPickBlock>(ord_key(best), k, L, tid, lane, wv);
    const float bound = key_to_float(bound_key);
    row_sweep<12>(xr, n, tid, wv, [&](int word, float v, bool in) {
        if (in && !(v < bound)) {
            const uint32_t key = ord_key(v);
            if (key >= bound_key) {
                const uint32_t at = atomicAdd(&L.cnt, 1u);
                if (at < (uint32_t)kPickList) L.list[at] = ((uint64_t)key << 32) | (uint32_t)~(word * kWave + lane);
            }
        }
    });
    __syncthreads();
    int cnt = (int)L.cnt;
    if (cnt < k || cnt > kPickList) cnt = pick_hard<kPickBlock, false>(xr, n, k, o, L, bound_key, cnt);
    emit_winners<kPickBlock, false>(L, cnt, k, o, tid);
}

// ---- neighbourhoods of heads whose candidate lists overflowed ------------------------
// The filter route (mfma_cosine.hip) gives up on a head when a candidate list cannot hold what
// reaches the bound (masses of equal edges, an adversarial key order) and raises the head's
// flag.  Such heads are rare, so they are not worth an [heads, S, P] edge block in memory: a
// fixed number of workgroups walk the (head, source) rows of the flagged heads, and each row's
// edges (Eq. 1) go to the workgroup's own scratch row of P floats, out of which the exact top-m
// (Eq. 3) is taken by the row kernels above.  The edges are formed exactly as in the streaming
// kernels -- the same matrix-core instruction sequence with the source in every operand row, the
// same norms -- so that a head gets the same bits whichever route it takes.
constexpr int kRedoBlock = 1024;
constexpr size_t kRedoLds = (size_t)(kRedoBlock / kWave) * kBlk * kPitch;   // a block of keys per wave

// Workgroups that walk the rows of flagged heads: one per compute unit, fewer for long rows
// (their scratch rows stay within 64 MiB), at least 16.
__host__ __device__ inline int redo_rows_workgroups(int heads, int S, int P)
{
    const long items = (long)heads * S;
    long wgs = ((long)64 << 20) / ((long)P * 4);
    wgs = wgs < 16 ? 16 : (wgs > 256 ? 256 : wgs);
    return (int)(items < wgs ? items : wgs);
}

struct RedoArgs {
    const uint16_t *Ac, *Kc;
    int N, P, S, m, heads;
    const int32_t *src, *overflow;
    float *rows;
    int32_t *nbr;
    float *nbr_e;
};

// Row `item` (head * S + source slot): its edges to the workgroup's scratch row, its m best to the lists.  mem: kRedoLds
// bytes.  Begins with a barrier.  A wave takes 32 keys at a time, fetched whole rows at a time and turned into operand
// layout in its own part of the LDS (operand layout straight from memory touches every line four times, and the waves'
// lines do not fit the first-level cache).  Whole calls, us, operand layout from memory and a radix selection / this way:
// 64 heads x 64 rows of 10000 keys 1438 / 770; key norms, clustered keys, two rounds: 8 heads of 32736 keys 460 / 294,
// 64 of 16352 526 / 438, 256 of 32736 9000 / 4895.  (The same in front of the kernel that takes the update along, with the
// general selection, which needs no more registers, and without a launch of its own: 338, 490 and 8300, and 104.3 instead
// of 105.4 for 8 heads of 16K keys with nothing to redo.)
__device__ __forceinline__ void redo_row(const RedoArgs &a, long item, unsigned char *mem)
{
    const int tid = here(threadIdx.x), lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5, h = (int)(item / a.S);
    float *erow = a.rows + (long)blockIdx.x * a.P;
    const int32_t i = a.src[item];
    const uint16_t *ah = a.Ac + (long)h * a.N * kD, *kh = a.Kc + (long)h * a.N * kD;
    unsigned char *tile = mem + wv * (kBlk * kPitch);
    __syncthreads();                          // the previous row's LDS and scratch row are free
    // the source's row in every row of the operand (a lane holds elements 16 s + 8 hh ..)
    bf16x8 q[kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) q[s] = load8(ah + (long)i * kD + 16 * s + 8 * hh);
    float sq_i = half_row_sumsq(q);
    sq_i = add_other_half(sq_i);
    const float inv_i = inv_norm(sq_i);
    // key l32 of a block is the operand's column
    for (int j0 = wv * kBlk; j0 < a.P; j0 += (kRedoBlock / kWave) * kBlk) {
        u32x4 piece[kSteps];
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int g = lane + kWave * u;   // 16 bytes: row g / 16 of the block
            const uint32_t at = (uint32_t)min(j0 + (g >> 4), a.P - 1) * (uint32_t)(2 * kD) + 16u * (g & 15);   // (below 4 GiB)
            piece[u] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(kh) + at);
        }
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int g = lane + kWave * u;
            *reinterpret_cast<u32x4 *>(tile + (g >> 4) * kPitch + 16 * (g & 15)) = piece[u];
        }
        wave_sync();
        f32x16 acc;
#pragma unroll
        for (int u = 0; u < 16; ++u) acc[u] = 0.f;
        float sq = 0.f;
        const unsigned char *mine = tile + l32 * kPitch + 16 * hh;
#pragma unroll
        for (int half = 0; half < 2; ++half) {   // (in two halves: registers)
            bf16x8 kc[kSteps / 2];
#pragma unroll
            for (int s = 0; s < kSteps / 2; ++s) kc[s] = *reinterpret_cast<const bf16x8 *>(mine + 32 * (half * (kSteps / 2) + s));
#pragma unroll
            for (int s = 0; s < kSteps / 2; ++s)   // rows = the source (32 times), columns = keys
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[half * (kSteps / 2) + s], kc[s], acc, 0, 0, 0);
            sq = half_row_sumsq(kc, sq);
            __builtin_amdgcn_sched_barrier(0);
        }
        sq = add_other_half(sq);
        const float e = (acc[0] * inv_norm(sq)) * inv_i;
        const int j = j0 + l32;
        if (hh == 0 && j < a.P) erow[j] = j == i ? -INFINITY : e;   // (Eq. 3: j != i)
        wave_sync();                          // the tile is read before the next block's rows go in
    }
    __syncthreads();                          // the row is complete and visible to the workgroup
    if (a.P <= 32 * kRedoBlock && a.m <= kSmallK) {
        PickLds<kRedoBlock> &L = *reinterpret_cast<PickLds<kRedoBlock> *>(mem);
        const PickOut o{a.m, a.nbr + item * a.m, nullptr, a.nbr_e + item * a.m};
        float val[32];
        load_row<kRedoBlock>(erow, a.P, tid, val);
        L.clear(tid);
        pick_row<kRedoBlock, 32, true, true>(val, erow, a.P, a.m, o, L, tid, lane, wv);
    } else {
        topk_stream_row<kRedoBlock, false>(0, erow, a.P, a.P, a.m, a.nbr + item * a.m, 0, a.nbr_e + item * a.m, 0, 0, 0, 0);
    }
}

__global__ __launch_bounds__(kRedoBlock) void redo_rows_kernel(RedoArgs a)
{
    extern __shared__ __align__(16) unsigned char mem[];
    int open = 0;   // any flagged head at all?  (a few loads instead of a walk over all rows)
    for (int g = threadIdx.x; g < a.heads; g += kRedoBlock) open |= a.overflow[g] != 0;
    if (!__syncthreads_or(open)) return;
    for (long item = blockIdx.x; item < (long)a.heads * a.S; item += gridDim.x)
        if (a.overflow[item / a.S]) redo_row(a, item, mem);   // (the same for every thread)
}

template <int ITEMS>   // 0: rows beyond 32768 entries
__global__ __launch_bounds__(kPickBlock) void pick_sources_kernel(
    const float *__restrict__ x, long ld, int n, int k, int S, int32_t *__restrict__ src_out, long src_ld,
    int32_t *__restrict__ ext_out, long ext_ld)
{
    __shared__ PickLds<kPickBlock> L;
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float *xr = x + (long)row * ld;
    const PickOut o{S, src_out + (long)row * src_ld, ext_out ? ext_out + (long)row * ext_ld : nullptr, nullptr};
    if constexpr (ITEMS > 0) {
        float val[ITEMS];
        load_row<kPickBlock>(xr, n, tid, val);
        L.clear(tid);
        pick_row<kPickBlock, ITEMS, false>(val, xr, n, k, o, L, tid, lane, wv);
    } else {
        pick_row_long(xr, n, k, o, L, tid, lane, wv);
    }
}

// A later round's sources and, in the same workgroup, the update of the round before and where the
// sources' lists come from (launches of their own cost 7.7 and 6.1 us with 8 heads).  The lists that the update reads are those that the match hands on.  (8 heads with 2048
// triples: 19.4 us for 32736 nodes and 17.0 for 15969 with the row read behind the update and the lists read again;
// 16.6 and 12.7 this way.)
template <int ITEMS, int D>
__global__ __launch_bounds__(kPickBlock) void pick_match_kernel(float *x, int n, MatchArgs a, int32_t *__restrict__ src_out,
                                                                DecayArgs update)
{
    static_assert(kPickBlock == kMatchBlock && kPickBlock == kUpdateBlock, "one workgroup does all");
    extern __shared__ __align__(16) unsigned char mem[];   // the update's, then the selection's
    PickLds<kPickBlock> &L = *reinterpret_cast<PickLds<kPickBlock> *>(mem);
    __shared__ int32_t match_lds[2 * kSmallK + kMaxExtSources], to_s[kSmallK];
    __shared__ int32_t wave_new[kPickBlock / kWave], wave_fb[kPickBlock / kWave];
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    float *xr = x + (long)h * n;
    int32_t *src = src_out + (long)h * a.S;
    const PickOut o{a.S, src, nullptr, nullptr};
    Triples<D> tri;
    bool bad;
    if constexpr (ITEMS == 0) {
        bad = match_load(a, h, match_lds, tid);
        pick_row_long(xr, n, a.S, o, L, tid, lane, wv);
    } else {
        // (what the match needs first, then the update, then the row: loads come back in the order they leave)
        const int32_t prev = a.prev_src[(long)h * a.S + min(tid, a.S - 1)];
        const int32_t spec = a.X > 0 ? a.ext[(long)h * (a.S + a.X) + a.S + min(tid, a.X - 1)] : 0;
        bad = a.X == 0 || (a.first ? a.overflow[h] : a.spec_bad[h]) != 0;
        tri.load(update, h, tid);
        float val[ITEMS];
        load_row<kPickBlock>(xr, n, here(threadIdx.x), val);
        const int tid = here(threadIdx.x), lane = tid & 63, wv = tid >> 6;
        if (a.X > 0 && a.first && tid == 0) a.spec_bad[h] = bad ? 1 : 0;
        if (tid < a.S) match_lds[tid] = prev;
        if (tid < a.X) match_lds[2 * a.S + tid] = spec;
        if (tid < kSmallK) to_s[tid] = -1;
        if constexpr (D > 0) update_row<ITEMS, D>(val, tri, xr, h, update, mem, tid);
        L.clear(tid);
        pick_row<kPickBlock, ITEMS, false>(val, xr, n, a.S, o, L, tid, lane, wv);
    }
    __syncthreads();   // the sources are written, the flag is read
    if (tid == 0) a.overflow[h] = 0;
    match_head<D>(a, h, bad, src, match_lds, to_s, wave_new, wave_fb, tri, tid);
}
template <int ITEMS, int D> constexpr size_t pick_match_lds()
{
    return update_row_lds<ITEMS, D>() > sizeof(PickLds<kPickBlock>) ? update_row_lds<ITEMS, D>() : sizeof(PickLds<kPickBlock>);
}

// The k best edges of each row of a dense edge block, ascending indices, with their values.
template <int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void pick_edges_kernel(const float *__restrict__ x, long ld, int n, int k,
                                                           int32_t *__restrict__ idx_out, long idx_ld,
                                                           float *__restrict__ val_out, long val_ld)
{
    __shared__ PickLds<BLOCK> L;
    const long row = blockIdx.x;
    const int tid = threadIdx.x;
    const PickOut o{k, idx_out + row * idx_ld, nullptr, val_out + row * val_ld};
    float val[ITEMS];
    load_row<BLOCK>(x + row * ld, n, tid, val);
    L.clear(tid);
    pick_row<BLOCK, ITEMS, true>(val, x + row * ld, n, k, o, L, tid, tid & 63, tid >> 6);
}

// ---- budgeted selection ---------------------------------------------------------------
// The B_l - w best entries of each row in ascending index order, then the window (Problem
// Formulation).  One workgroup of 16 waves per row; what bounds it is the chain of steps, each a
// round trip to memory or LDS, so the steps are few: the row's keys sit in registers, one histogram
// sweep over 11 bits of key - kmin finds the bin of the cut, the bin's entries (usually below a
// hundred) go to a list on which every thread ranks one entry against all others, and the
// winners' places come from wave votes and one scan of the vote counts.  All scans run on the
// vector ALU (common.hpp).  (Three histogram sweeps through LDS copies of the keys, with a
// one-wave bin search whose lanes all hit the same LDS bank: 27.6 us for 8 rows of 32736 entries;
// this way 15.2 us; 256 threads and two
// histogram sweeps more: 13.9 us for rows of 4064 entries, this way 5.6 us.)
constexpr int kBudgetBlock = 1024;
constexpr int kBudgetList = 8192;    // entries in the cut's bin that the long-row kernel can list
constexpr int kPairs = 1024;         // ... that are ranked pair by pair

// Which of the `cnt` (<= kPairs) listed keys is the need-th largest: out[0] = that key, out[1] =
// how many entries equal to it are among the need largest, out[2] = how many there are.  `list` is
// padded with zeros (below every key) to a multiple of four.  Ends with a barrier.
__device__ __forceinline__ void rank_in_pairs(const uint32_t *list, int cnt, uint32_t need, uint32_t *out, int tid)
{
    if (tid < cnt) {
        const uint32_t mine = list[tid];
        uint32_t above = 0, same = 0;
        for (int u = 0; u < cnt; u += 4) {
            const uint4 o = *reinterpret_cast<const uint4 *>(list + u);
            above += (o.x > mine) + (o.y > mine) + (o.z > mine) + (o.w > mine);
            same += (o.x == mine) + (o.y == mine) + (o.z == mine) + (o.w == mine);
        }
        if (above < need && need <= above + same) {   // (every entry equal to the cut writes the same)
            out[0] = mine;
            out[1] = need - above;
            out[2] = same;
        }
    }
    __syncthreads();
}

// The need-th largest of the cnt <= kBudgetList listed keys (padded with zeros to a multiple of four where
// cnt <= kPairs): tau = that key, need = how many entries equal to it are among the need largest, equal =
// how many there are.  false if many ties straddle the cut.  Every thread calls it and gets the same; `hist`,
// `part` and `out` are free.
__device__ __forceinline__ bool cut_of_list(const uint32_t *lkey, uint32_t cnt, uint32_t &need, uint32_t &tau,
                                            uint32_t &equal, uint32_t *hist, uint32_t *part, uint32_t *out, int tid,
                                            int lane, int wv)
{
    if (cnt <= (uint32_t)kPairs) {
        rank_in_pairs(lkey, (int)cnt, need, out, tid);
        tau = out[0];
        need = out[1];
        equal = out[2];
        return true;
    }
    tau = 0u;                            // radix select over the listed keys, 11 bits a sweep
    equal = cnt;
    for (int left = 32; left > 0;) {
        const int low = left > 11 ? left - 11 : 0;
        hist[tid] = 0;
        hist[tid + kBudgetBlock] = 0;
        __syncthreads();
        for (int r = tid; r < (int)cnt; r += kBudgetBlock) {
            const uint32_t key = lkey[r];
            if (left == 32 || (key >> left) == (tau >> left)) atomicAdd(&hist[(key >> low) & 2047u], 1u);
        }
        __syncthreads();
        find_bin_block<kBudgetBlock>(hist, need, part, out, tid, lane, wv);
        tau |= out[0] << low;
        need = out[1];
        equal = out[2];
        left = low;
        __syncthreads();
    }
    return equal == need;
}

// Whether entry r of the list is among the winners that cut_of_list() cut off: of the entries equal to the
// cut the `need` with the lowest indices are.
__device__ __forceinline__ bool list_wins(const uint32_t *lkey, const uint32_t *lidx, uint32_t cnt, int r, uint32_t tau,
                                          uint32_t need, uint32_t equal)
{
    const uint32_t key = lkey[r], j = lidx[r];
    if (key != tau || equal == need) return key >= tau;
    uint32_t rank = 0;
    for (int u = 0; u < (int)cnt; ++u) rank += lkey[u] == tau && lidx[u] < j;
    return rank < need;
}

// Indices of the k set bits of a bitmap in LDS -> out, ascending.  A thread owns a run of words: it
// counts their bits, one scan over the workgroup places the run, and it writes the run's indices.  A bitmap
// with another number of bits is left alone (false, the same for every thread).
template <int NW>
__device__ __forceinline__ bool emit_bitmap(const uint64_t *map, int words, int k, uint32_t *part, int32_t *out, int tid,
                                            int lane, int wv)
{
    const int per = (words + NW * kWave - 1) / (NW * kWave), w0 = min(tid * per, words), w1 = min(w0 + per, words);
    uint32_t mine = 0, total;
    for (int w = w0; w < w1; ++w) mine += (uint32_t)__popcll(map[w]);
    int32_t *o = out + block_scan_add<NW>(mine, part, lane, wv, total);
    if (total != (uint32_t)k) return false;
    for (int w = w0; w < w1; ++w) {
        uint64_t bits = map[w];
        while (bits) {
            *o++ = w * kWave + __ffsll((long long)bits) - 1;
            bits &= bits - 1;
        }
    }
    return true;
}

struct BudgetLds {
    __align__(16) uint32_t hist[2 * kBudgetBlock];
    __align__(16) uint32_t list[kPairs];
    uint32_t part[2][kBudgetBlock / kWave], lo[kBudgetBlock / kWave], hi[kBudgetBlock / kWave], out[3], cnt;
    uint64_t map[1];   // ITEMS * 16 words
};
template <int ITEMS, int D> constexpr size_t budget_lds()
{
    const size_t own = sizeof(BudgetLds) + (size_t)ITEMS * (kBudgetBlock / kWave) * 8;
    return update_row_lds<ITEMS, D>() > own ? update_row_lds<ITEMS, D>() : own;
}

// The k best of a row held in registers, ascending indices -> out.
template <int ITEMS>
__device__ __forceinline__ void budget_row(const float (&row)[ITEMS], int n, int k, int32_t *out, BudgetLds &L, int tid,
                                           int lane, int wv)
{
    constexpr int NW = kBudgetBlock / kWave, CELLS = ITEMS * NW;
    uint32_t *hist = L.hist, *list = L.list, *s_out = L.out;
    uint64_t *map = L.map;
    float val[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) val[i] = row[i];
    hist[tid] = 0;
    hist[tid + kBudgetBlock] = 0;
    list[tid] = 0;
    if (tid == 0) L.cnt = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) asm volatile("" : "+v"(val[i]));   // (the batch of loads stays one)
    uint32_t key[ITEMS], kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool in = i * kBudgetBlock + tid < n;
        key[i] = in ? entry_key(val[i]) : 0u;
        kmin = min(kmin, in ? key[i] : 0xffffffffu);
        kmax = max(kmax, key[i]);
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { L.lo[wv] = kmin; L.hi[wv] = kmax; }
    __syncthreads();
    kmin = wave_min_u32(L.lo[lane & (NW - 1)]);
    kmax = wave_max_u32(L.hi[lane & (NW - 1)]);

    // radix select on key - kmin from the top bit in which the row's keys differ; it ends when the
    // bin of the cut is one key wide or holds few enough entries to rank them pair by pair
    int shift = kmax > kmin ? 32 - __clz(kmax - kmin) : 0;
    uint32_t tau = kmin, need = (uint32_t)k, equal = (uint32_t)n;
    for (int sweep = 0; shift > 0; ++sweep) {
        const int below = shift;   // key bits that may still differ inside the current bin
        shift = below > 11 ? below - 11 : 0;
        const uint32_t width = below < 32 ? (1u << below) - 1u : 0xffffffffu;   // of the current bin, less one
        if (sweep > 0) {
            hist[tid] = 0;
            hist[tid + kBudgetBlock] = 0;
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (key[i] >= tau && key[i] - tau <= width) atomicAdd(&hist[(key[i] - tau) >> shift], 1u);
        __syncthreads();
        find_bin_block<kBudgetBlock>(hist, need, L.part[0], s_out, tid, lane, wv);
        tau += s_out[0] << shift;
        need = s_out[1];
        equal = s_out[2];
        if (shift > 0 && equal <= (uint32_t)kPairs) {
            const uint32_t bin = (1u << shift) - 1u;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (key[i] - tau <= bin) list[atomicAdd(&L.cnt, 1u)] = key[i];   // (lower keys wrap around, bin < 2^21)
            __syncthreads();   // (also: s_out is read by every thread)
            rank_in_pairs(list, (int)equal, need, s_out, tid);
            tau = s_out[0];
            need = s_out[1];
            equal = s_out[2];
            break;
        }
        __syncthreads();       // s_out and the histogram are read before the next sweep writes them
    }

    // Winners: every key above tau and the `need` first of those equal to it.  Entry i of thread
    // tid has index i * 1024 + tid, so the vote on entry i of wave wv is word i * 16 + wv of a
    // bitmap of the row.  The ties that stay out leave it again, last index first.
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint64_t in = __ballot(key[i] >= tau);
        if (lane == 0) map[i * NW + wv] = in;
    }
    __syncthreads();
    if (equal != need) {
        // rank of each tied entry in index order: votes per word, one scan over the words
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint64_t eq = __ballot(key[i] == tau);
            if (lane == 0) hist[i * NW + wv] = (uint32_t)__popcll(eq);
        }
        __syncthreads();
        uint32_t total;
        const uint32_t before = block_scan_add<NW>(tid < CELLS ? hist[tid] : 0u, L.part[0], lane, wv, total);
        if (tid < CELLS) hist[tid] = before;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint64_t eq = __ballot(key[i] == tau);
            const uint64_t drop = __ballot(key[i] == tau && hist[i * NW + wv] + votes_below(eq) >= need);
            if (lane == 0) map[i * NW + wv] &= ~drop;
        }
        __syncthreads();
    }
    (void)emit_bitmap<NW>(map, min(CELLS, (n + kWave - 1) / kWave), k, L.part[1], out, tid, lane, wv);
}

template <int ITEMS, int D>
__global__ __launch_bounds__(kBudgetBlock) void budget_select_kernel(
    float *x, int n, int32_t *__restrict__ idx_out, int append_from, int append_count, DecayArgs update, GatherArgs rows,
    LayerPlan plan)
{
    static_assert(kBudgetBlock == kUpdateBlock, "one workgroup does both");
    extern __shared__ __align__(16) unsigned char mem[];   // the update's, then the selection's
    BudgetLds &L = *reinterpret_cast<BudgetLds *>(mem);
    const int row = blockIdx.x;
    const int g = row / plan.heads_per_layer, hl = row % plan.heads_per_layer;
    const int k = plan.budget[g] - append_count;
    int32_t *out = idx_out + (plan.row_off[g] + (long)hl * plan.budget[g]);
    float *xr = x + (long)row * n;
    Triples<D> tri;
    tri.load(update, row, threadIdx.x);
    float val[ITEMS];
    load_row<kBudgetBlock>(xr, n, here(threadIdx.x), val);
    const int tid = here(threadIdx.x), lane = tid & 63, wv = tid >> 6;
    for (int r = tid; r < append_count; r += kBudgetBlock) out[k + r] = append_from + r;
    if constexpr (D > 0) update_row<ITEMS, D>(val, tri, xr, row, update, mem, tid);   // (the last round's, in a whole pass)
    budget_row<ITEMS>(val, n, k, out, L, tid, lane, wv);
    if (!rows.Kout) return;
    // The retained rows of K and V, 16 bytes a thread: with little to copy that is done before a launch of its own
    // would have begun.
    __syncthreads();   // the indices are written
    const int pieces = rows.row_bytes / 16, B = k + append_count;
    const long from0 = (long)row * rows.N, to0 = (plan.row_off[g] + (long)hl * plan.budget[g]) * pieces;
    for (int u = tid; u < B * pieces; u += kBudgetBlock) {
        const long from = (from0 + out[u / pieces]) * pieces + u % pieces;
        const uint4 a = ((const uint4 *)rows.Kc)[from], b = ((const uint4 *)rows.Vc)[from];
        ((uint4 *)rows.Kout)[to0 + u] = a;
        ((uint4 *)rows.Vout)[to0 + u] = b;
    }
}

// Rows beyond 32768 entries: two reads instead of five.  A coarse sample gives the key range, the
// first read counts every key into 2048 bins over it (keys outside go to the end bins: bins only
// have to be monotone), the second marks the entries of higher bins in a bitmap in LDS and lists those
// of the cut's bin, whose winners join the bitmap; the indices are then read off the bitmap in
// order.  Bound by the vector instructions of one compute unit (a row of 131008 entries is 512
// wave-wide entries per SIMD, four clocks an instruction): the first read takes nine per entry, the
// second, which compares the floats with the ends of the bin, about five.  A row with more than
// kBudgetList entries in the bin of the cut (masses of equal values), or with more ties at the cut
// than can be ranked pair by pair, goes through the general algorithm.  (Five reads with an LDS
// histogram of 11, 11 and 10 bits: 110 us for 8 rows of 131008 entries; this way 33 us.)
__global__ __launch_bounds__(kBudgetBlock) void budget_select_long_kernel(
    const float *__restrict__ x, int n, int32_t *__restrict__ idx_out, int append_from, int append_count, LayerPlan plan)
{
    constexpr int NW = kBudgetBlock / kWave, SAMPLE = 4;
    extern __shared__ __align__(16) uint32_t dyn[];
    __shared__ __align__(16) uint32_t hist[2 * kBudgetBlock];
    __shared__ uint32_t s_part[2][NW], s_min[NW], s_max[NW], s_out[3], s_cnt;
    const int words = (n + kWave - 1) / kWave;
    uint32_t *lkey = dyn, *lidx = dyn + kBudgetList;                                // the cut's bin
    uint64_t *map = reinterpret_cast<uint64_t *>(dyn + 2 * kBudgetList);            // [words] bit l of word w: entry 64 w + l is in
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int g = row / plan.heads_per_layer, hl = row % plan.heads_per_layer;
    const int k = plan.budget[g] - append_count;
    int32_t *out = idx_out + (plan.row_off[g] + (long)hl * plan.budget[g]);
    const float *xr = x + (long)row * n;

    // range of the sample: SAMPLE stretches of 64 entries per wave, evenly spread
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    {
        float v[SAMPLE];
#pragma unroll
        for (int i = 0; i < SAMPLE; ++i)
            v[i] = xr[(int)((long)(i * NW + wv) * (words - 1) / (SAMPLE * NW)) * kWave + lane];
        hist[tid] = 0;
        hist[tid + kBudgetBlock] = 0;
        if (tid == 0) s_cnt = 0;
        for (int r = tid; r < append_count; r += kBudgetBlock) out[k + r] = append_from + r;
#pragma unroll
        for (int i = 0; i < SAMPLE; ++i) {
            const uint32_t key = ord_key(v[i]);
            kmin = min(kmin, key);
            kmax = max(kmax, key);
        }
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { s_min[wv] = kmin; s_max[wv] = kmax; }
    __syncthreads();
    kmin = wave_min_u32(s_min[lane & (NW - 1)]);
    kmax = wave_max_u32(s_max[lane & (NW - 1)]);
    const int bits = kmax > kmin ? 32 - __clz(kmax - kmin) : 0, shift = bits > 11 ? bits - 11 : 0;
    row_sweep<16>(xr, n, tid, wv, [&](int, float v, bool in) {
        if (in) atomicAdd(&hist[(min(max(ord_key(v), kmin), kmax) - kmin) >> shift], 1u);
    });
    __syncthreads();
    find_bin_block<kBudgetBlock>(hist, (uint32_t)k, s_part[0], s_out, tid, lane, wv);
    const uint32_t bin = s_out[0], cnt = s_out[2];
    uint32_t need = s_out[1];
    if (cnt > (uint32_t)kBudgetList) {   // (the same for every thread)
        topk_stream_row<kBudgetBlock, true>(row, x, n, n, 0, idx_out, 0, nullptr, 0, append_from, append_count, plan);
        return;
    }
    if (tid < 4) lkey[min(cnt + (uint32_t)tid, (uint32_t)kBudgetList - 1u)] = 0u;   // padding for reads of four
    __syncthreads();
    // The floats at the ends of the bin (the end bins are open).  Floats compare as their keys do, but for
    // two: the key below +0.0 stands for no number and reads back as -0.0, which +0.0 does not exceed (the
    // number below it ends the bin instead), and NaN compares with nothing.
    const uint32_t last_bin = (kmax - kmin) >> shift, top = kmin + (bin << shift) + ((1u << shift) - 1u);
    const float flo = bin == 0 ? -INFINITY : key_to_float(kmin + (bin << shift));
    const float fhi = bin == last_bin ? INFINITY : key_to_float(top == 0x7fffffffu ? top - 1u : top);
    row_sweep<16>(xr, n, tid, wv, [&](int word, float v, bool in) {
        const bool reach = in && v >= flo, over = reach && v > fhi;
        const uint64_t above = __ballot(over);
        if (lane == 0 && word < words) map[word] = above;
        if (reach && !over) {
            const uint32_t at = atomicAdd(&s_cnt, 1u);
            if (at < (uint32_t)kBudgetList) {
                lkey[at] = ord_key(v);
                lidx[at] = (uint32_t)(word * kWave + lane);
            }
        }
    });
    __syncthreads();
    if (s_cnt != cnt) {   // counted by key, not found by comparison: NaN in the bin
        topk_stream_row<kBudgetBlock, true>(row, x, n, n, 0, idx_out, 0, nullptr, 0, append_from, append_count, plan);
        return;
    }
    // the need-th largest of the list
    uint32_t tau, equal;
    if (!cut_of_list(lkey, cnt, need, tau, equal, hist, s_part[1], s_out, tid, lane, wv)) {
        topk_stream_row<kBudgetBlock, true>(row, x, n, n, 0, idx_out, 0, nullptr, 0, append_from, append_count, plan);
        return;
    }
    for (int r = tid; r < (int)cnt; r += kBudgetBlock) {
        const uint32_t j = lidx[r];
        if (list_wins(lkey, lidx, cnt, r, tau, need, equal))
            atomicOr(reinterpret_cast<uint32_t *>(map) + (j >> 5), 1u << (j & 31u));
    }
    __syncthreads();
    if (!emit_bitmap<NW>(map, words, k, s_part[0], out, tid, lane, wv))   // NaN counted above the bin and not marked
        topk_stream_row<kBudgetBlock, true>(row, x, n, n, 0, idx_out, 0, nullptr, 0, append_from, append_count, plan);
}

// Few long rows: a row's entries are shared out to workgroups of kSegment entries, in two launches.  One
// compute unit alone spends its time on the row's vector instructions and LDS atomics (131072 entries are 512
// wave-wide entries per SIMD, each a dozen instructions over two reads).  The first launch counts a segment's
// keys into 2048 bins over the range of a coarse sample of the row (the same in every workgroup of a row; keys
// outside go to the end bins) and sorts its entries by bin.  In the second, every workgroup adds up the row's
// counts, finds the bin of the cut, fetches that bin's entries from all segments (they lie side by side in
// each), cuts them as above, and writes the winners of its own segment: their places start behind the winners
// of the segments before it, which the counts and the list give.  A row whose cut falls among too many equal
// or nearly equal values goes through the general algorithm, by its first workgroup.  What is left is two launches
// and their chains of loads.  (8 rows of 131008 entries: 32.8 us with one workgroup a row, 12.3 us this way.)
constexpr int kSegment = 8 * kBudgetBlock;
constexpr int kMaxSegments = 32;

struct SplitScratch {
    uint4 *range;      // [rows] kmin, kmax, shift of the bins
    uint16_t *above;   // [rows, segments, 2048] entries of the segment in higher bins
    uint16_t *order;   // [rows, segments, kSegment] places in the segment, highest bin first
};

__global__ __launch_bounds__(kBudgetBlock) void split_count_kernel(const float *__restrict__ x, int n, SplitScratch sc)
{
    constexpr int NW = kBudgetBlock / kWave, SAMPLE = 4, ITEMS = kSegment / kBudgetBlock;
    __shared__ __align__(16) uint32_t hist[2 * kBudgetBlock];
    __shared__ __align__(16) uint16_t order[kSegment];
    __shared__ uint32_t s_part[NW], s_min[NW], s_max[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x, seg = blockIdx.y;
    const int words = (n + kWave - 1) / kWave, base = seg * kSegment;
    const float *xr = x + (long)row * n;
    float v[SAMPLE], val[ITEMS];
#pragma unroll
    for (int i = 0; i < SAMPLE; ++i)   // stretches of 64 entries, evenly spread
        v[i] = xr[(int)((long)(i * NW + wv) * (words - 1) / (SAMPLE * NW)) * kWave + lane];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) val[i] = xr[min(base + i * kBudgetBlock + tid, n - 1)];
    hist[tid] = 0;
    hist[tid + kBudgetBlock] = 0;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int i = 0; i < SAMPLE; ++i) {
        const uint32_t key = ord_key(v[i]);
        kmin = min(kmin, key);
        kmax = max(kmax, key);
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { s_min[wv] = kmin; s_max[wv] = kmax; }
    __syncthreads();
    kmin = wave_min_u32(s_min[lane & (NW - 1)]);
    kmax = wave_max_u32(s_max[lane & (NW - 1)]);
    const int bits = kmax > kmin ? 32 - __clz(kmax - kmin) : 0, shift = bits > 11 ? bits - 11 : 0;
    if (seg == 0 && tid == 0) sc.range[row] = make_uint4(kmin, kmax, (uint32_t)shift, 0u);
    uint32_t bin[ITEMS], at[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        bin[i] = (min(max(ord_key(val[i]), kmin), kmax) - kmin) >> shift;
        at[i] = base + i * kBudgetBlock + tid < n ? atomicAdd(&hist[bin[i]], 1u) : 0u;
    }
    __syncthreads();
    // thread t owns two bins, the highest pair first
    const int hi = 2 * (kBudgetBlock - 1 - tid);
    const uint2 c = *reinterpret_cast<const uint2 *>(hist + hi);
    uint32_t total;
    const uint32_t higher = block_scan_add<NW>(c.x + c.y, s_part, lane, wv, total);
    *reinterpret_cast<uint2 *>(hist + hi) = make_uint2(higher + c.y, higher);
    const long part = (long)row * gridDim.y + seg;
    reinterpret_cast<uint32_t *>(sc.above + part * 2 * kBudgetBlock)[hi >> 1] = (higher + c.y) | higher << 16;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (base + i * kBudgetBlock + tid < n) order[hist[bin[i]] + at[i]] = (uint16_t)(i * kBudgetBlock + tid);
    __syncthreads();
    // (behind the row's end: whatever the LDS holds, never read)
    reinterpret_cast<uint4 *>(sc.order + part * kSegment)[tid] = reinterpret_cast<const uint4 *>(order)[tid];
}

__global__ __launch_bounds__(kBudgetBlock) void split_select_kernel(
    const float *__restrict__ x, int n, int32_t *__restrict__ idx_out, int append_from, int append_count, SplitScratch sc,
    LayerPlan plan)
{
    constexpr int NW = kBudgetBlock / kWave, ITEMS = kSegment / kBudgetBlock, BINS = 2 * kBudgetBlock;
    extern __shared__ __align__(16) uint32_t dyn[];
    __shared__ __align__(16) uint32_t hist[BINS];
    __shared__ uint64_t map[kSegment / kWave];
    __shared__ uint32_t s_part[2][NW], s_out[3], s_off[kMaxSegments], s_end[kMaxSegments], s_base[kMaxSegments], s_before;
    uint32_t *lkey = dyn, *lidx = dyn + kBudgetList;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x, seg = blockIdx.y, segs = gridDim.y;
    const int g = row / plan.heads_per_layer, hl = row % plan.heads_per_layer, base = seg * kSegment;
    const int k = plan.budget[g] - append_count;
    int32_t *out = idx_out + (plan.row_off[g] + (long)hl * plan.budget[g]);
    const float *xr = x + (long)row * n;
    const uint16_t *above = sc.above + (long)row * segs * BINS;
    const uint4 range = sc.range[row];
    float val[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) val[i] = xr[min(base + i * kBudgetBlock + tid, n - 1)];
    // the row's entries above each bin: thread t owns bins 2 t and 2 t + 1
    uint32_t lo = 0, hi = 0;
    for (int s0 = 0; s0 < segs; s0 += 8) {   // (the loads of eight segments leave together)
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = reinterpret_cast<const uint32_t *>(above + (long)min(s0 + u, segs - 1) * BINS)[tid];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < segs) { lo += v[u] & 0xffffu; hi += v[u] >> 16; }
    }
    hist[2 * tid] = lo;
    hist[2 * tid + 1] = hi;
    __syncthreads();
    const uint32_t below = tid ? hist[2 * tid - 1] : (uint32_t)n, need_k = (uint32_t)k;
    if (lo < need_k && need_k <= below) { s_out[0] = 2 * tid; s_out[1] = need_k - lo; s_out[2] = below - lo; }
    if (hi < need_k && need_k <= lo) { s_out[0] = 2 * tid + 1; s_out[1] = need_k - hi; s_out[2] = lo - hi; }
    __syncthreads();
    const uint32_t bin = s_out[0], cnt = s_out[2];
    uint32_t need = s_out[1];
    auto general = [&] {
        if (seg == 0)
            topk_stream_row<kBudgetBlock, true>(row, x, n, n, 0, idx_out, 0, nullptr, 0, append_from, append_count, plan);
    };
    if (cnt > (uint32_t)kBudgetList) {   // (the same for every thread and workgroup of the row)
        general();
        return;
    }
    if (wv == 0) {   // where the bin's entries lie in every segment and in the list, and the winners above it before this one
        const int s = min(lane, segs - 1);
        const uint32_t o = above[(long)s * BINS + bin];
        const uint32_t e = bin ? above[(long)s * BINS + bin - 1] : (uint32_t)min(kSegment, n - s * kSegment);
        const uint32_t here = lane < segs ? e - o : 0u, incl = wave_scan_add(here);
        const uint32_t before = wave_sum_u32(lane < seg ? o : 0u);
        if (lane < segs) { s_off[lane] = o; s_end[lane] = e; s_base[lane] = incl - here; }
        if (lane == 0) s_before = before;
    }
    if (tid < 4) lkey[min(cnt + (uint32_t)tid, (uint32_t)kBudgetList - 1u)] = 0u;   // padding for reads of four
    __syncthreads();
    for (int s = wv; s < segs; s += NW) {
        const uint16_t *o = sc.order + ((long)row * segs + s) * kSegment;
        for (uint32_t l = s_off[s] + lane; l < s_end[s]; l += kWave) {
            const int j = s * kSegment + o[l];
            const uint32_t to = s_base[s] + l - s_off[s];
            lkey[to] = ord_key(xr[j]);
            lidx[to] = (uint32_t)j;
        }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool in = base + i * kBudgetBlock + tid < n;
        const uint32_t b = (min(max(ord_key(val[i]), range.x), range.y) - range.x) >> range.z;
        const uint64_t over = __ballot(in && b > bin);
        if (lane == 0) map[i * NW + wv] = over;
    }
    __syncthreads();
    uint32_t tau, equal;
    if (!cut_of_list(lkey, cnt, need, tau, equal, hist, s_part[1], s_out, tid, lane, wv)) {
        general();
        return;
    }
    for (int r = tid; r < (int)cnt; r += kBudgetBlock) {
        const int j = (int)lidx[r];
        if (j < base + kSegment && list_wins(lkey, lidx, cnt, r, tau, need, equal)) {
            if (j < base) atomicAdd(&s_before, 1u);
            else atomicOr(reinterpret_cast<uint32_t *>(map) + ((j - base) >> 5), 1u << (j & 31));
        }
    }
    __syncthreads();
    // a thread writes the winners among eight neighbours
    uint32_t eight = reinterpret_cast<const uint8_t *>(map)[tid], total;
    int32_t *o = out + s_before + block_scan_add<NW>((uint32_t)__popc(eight), s_part[0], lane, wv, total);
    for (int j = base + 8 * tid; eight; eight >>= 1, ++j)
        if (eight & 1u) *o++ = j;
    if (seg == 0)
        for (int r = tid; r < append_count; r += kBudgetBlock) out[k + r] = append_from + r;
}

template <int BLOCK, int DIG>
static hipError_t launch_lds(const float *x, long ld, int n, int rows, int k, int32_t *idx_out, long idx_ld,
                             float *val_out, long val_ld, hipStream_t st)
{
    const int items = (n + BLOCK - 1) / BLOCK;
    const size_t lds = ((size_t)items * BLOCK + 2 * (size_t)items * (BLOCK / kWave)) * 4;
    if (lds > 65536 && !allow_big_lds((const void *)topk_rows_lds_kernel<BLOCK, DIG>, 140 * 1024)) return hipGetLastError();
    hipLaunchKernelGGL((topk_rows_lds_kernel<BLOCK, DIG>), dim3(rows), dim3(BLOCK), lds, st, x, ld, n, k, idx_out, idx_ld,
                       val_out, val_ld);
    return hipGetLastError();
}

static hipError_t launch_pick(const float *x, long ld, int n, int rows, int k, int S, int32_t *src, long src_ld,
                              int32_t *ext, long ext_ld, hipStream_t st)
{
#define GKV_PICK(ITEMS) \
    hipLaunchKernelGGL(pick_sources_kernel<ITEMS>, dim3(rows), dim3(kPickBlock), 0, st, x, ld, n, k, S, src, src_ld, ext, ext_ld)
    if (n <= 1024) GKV_PICK(1);
    else if (n <= 2048) GKV_PICK(2);
    else if (n <= 4096) GKV_PICK(4);
    else if (n <= 8192) GKV_PICK(8);
    else if (n <= 16384) GKV_PICK(16);
    else if (n <= 32768) GKV_PICK(32);
    else GKV_PICK(0);
#undef GKV_PICK
    return hipGetLastError();
}

bool pick_match_applies(int S) { return S <= kSmallK; }

constexpr int kBigLds = 147456;   // dynamic LDS of the kernels that take an update along, at most
static_assert(update_row_lds<32, 2>() <= kBigLds && update_row_lds<32, 4>() <= kBigLds, "");

template <int D>
static hipError_t launch_pick_match_d(float *x, int n, int rows, const MatchArgs &a, int32_t *src,
                                      const DecayArgs &update, hipStream_t st)
{
#define GKV_PICK(ITEMS)                                                                                          \
    do {                                                                                                         \
        if (D > 0 && !allow_big_lds((const void *)pick_match_kernel<ITEMS, D>, kBigLds)) return hipGetLastError(); \
        hipLaunchKernelGGL((pick_match_kernel<ITEMS, D>), dim3(rows), dim3(kPickBlock), (pick_match_lds<ITEMS, D>()), st, x, n, \
                           a, src, update);                                                                      \
    } while (0)
    if (n <= 4096) GKV_PICK(4);   // (lists are kept on the filter route only: 2048 nodes or more)
    else if (n <= 8192) GKV_PICK(8);
    else if (n <= 16384) GKV_PICK(16);
    else if (n <= 32768) GKV_PICK(32);
    else if constexpr (D == 0) GKV_PICK(0);
    else return hipErrorInvalidValue;
#undef GKV_PICK
    return hipGetLastError();
}

hipError_t launch_pick_match(float *x, int n, int rows, const MatchArgs &a, int32_t *src, const DecayArgs &update,
                             hipStream_t st)
{
    if (a.S > kSmallK || a.X > kMaxExtSources) return hipErrorInvalidValue;
    switch (update.items) {
        case 0: return launch_pick_match_d<0>(x, n, rows, a, src, update, st);
        case 1: return launch_pick_match_d<1>(x, n, rows, a, src, update, st);
        case 2: return launch_pick_match_d<2>(x, n, rows, a, src, update, st);
        case 4: return launch_pick_match_d<4>(x, n, rows, a, src, update, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_topk_rows(const float *x, long ld, int n, int rows, int k, int32_t *idx_out, long idx_ld,
                            float *val_out, long val_ld, hipStream_t st)
{
    if (rows <= 0) return hipSuccess;
    if (k <= kSmallK && !val_out) return launch_pick(x, ld, n, rows, k, k, idx_out, idx_ld, nullptr, 0, st);
    if (k <= kSmallK && n <= 32768) {
#define GKV_EDGES(BLOCK, ITEMS)                                                                                  \
    hipLaunchKernelGGL((pick_edges_kernel<BLOCK, ITEMS>), dim3(rows), dim3(BLOCK), 0, st, x, ld, n, k, idx_out, idx_ld, \
                       val_out, val_ld)
        if (n <= 512) GKV_EDGES(256, 2);
        else if (n <= 1024) GKV_EDGES(256, 4);
        else if (n <= 2048) GKV_EDGES(256, 8);
        else if (n <= 4096) GKV_EDGES(256, 16);
        else if (n <= 8192) GKV_EDGES(256, 32);
        else if (n <= 16384) GKV_EDGES(1024, 16);
        else GKV_EDGES(1024, 32);
#undef GKV_EDGES
        return hipGetLastError();
    }
    if (n <= 4096) return launch_lds<256, 8>(x, ld, n, rows, k, idx_out, idx_ld, val_out, val_ld, st);
    if (n <= 32768) return launch_lds<1024, 11>(x, ld, n, rows, k, idx_out, idx_ld, val_out, val_ld, st);
    hipLaunchKernelGGL((topk_rows_stream_kernel<1024, false>), dim3(rows), dim3(1024), 0, st, x, ld, n, k, idx_out, idx_ld,
                       val_out, val_ld, 0, 0, 0);
    return hipGetLastError();
}

size_t redo_rows_scratch_bytes(int heads, int S, int P)
{
    return (size_t)redo_rows_workgroups(heads, S, P) * P * sizeof(float);
}

hipError_t launch_redo_rows(const void *Ac, const void *Kc, int heads, int N, int P, int S, int m, const int32_t *src,
                            const int32_t *overflow, float *rows, int32_t *nbr, float *nbr_e, hipStream_t st)
{
    const RedoArgs a{(const uint16_t *)Ac, (const uint16_t *)Kc, N, P, S, m, heads, src, overflow, rows, nbr, nbr_e};
    if (!allow_big_lds((const void *)redo_rows_kernel, (int)kRedoLds)) return hipGetLastError();
    hipLaunchKernelGGL(redo_rows_kernel, dim3(redo_rows_workgroups(heads, S, P)), dim3(kRedoBlock), kRedoLds, st, a);
    return hipGetLastError();
}

hipError_t launch_pick_sources(const float *x, long ld, int n, int rows, int S, int X, int32_t *src,
                               int32_t *ext, hipStream_t st)
{
    if (rows <= 0) return hipSuccess;
    if (S + X > n || S + X > kSmallK) return hipErrorInvalidValue;
    return launch_pick(x, ld, n, rows, S + X, S, src, S, ext, S + X, st);
}

// Row length up to which the budgeted selection keeps a bitmap of the row in LDS.
constexpr int kBitmapRow = 1 << 18;
static_assert(kBitmapRow <= kMaxSegments * kSegment, "segments of a row");

template <int D>
static hipError_t launch_budget_d(float *scores, int P, int rows, const LayerPlan &plan, int w, int32_t *idx,
                                  const DecayArgs &update, const GatherArgs &gather, hipStream_t st)
{
#define GKV_BUDGET(ITEMS)                                                                                       \
    do {                                                                                                        \
        if (D > 0 && !allow_big_lds((const void *)budget_select_kernel<ITEMS, D>, kBigLds)) return hipGetLastError(); \
        hipLaunchKernelGGL((budget_select_kernel<ITEMS, D>), dim3(rows), dim3(kBudgetBlock), (budget_lds<ITEMS, D>()), st, \
                           scores, P, idx, P, w, update, gather, plan);                                         \
    } while (0)
    if (P <= 1024) GKV_BUDGET(1);
    else if (P <= 2048) GKV_BUDGET(2);
    else if (P <= 4096) GKV_BUDGET(4);
    else if (P <= 8192) GKV_BUDGET(8);
    else if (P <= 16384) GKV_BUDGET(16);
    else GKV_BUDGET(32);
#undef GKV_BUDGET
    return hipGetLastError();
}

// Segments of a row that is shared out (0: it is not): rows longer than the kernels that hold one in registers
// take, up to the longest with a bitmap in LDS, as long as there are no more workgroups than compute units, or
// twice as many from eight segments on (us, one workgroup a row / split: 8 rows of 40000 entries 16.6 / 11.9,
// 64 17.1 / 18.3; 8 of 131008 32.8 / 12.3, 32 33.7 / 22.4, 64 34.5 / 41.2; 16 of 262144 56.6 / 25.0).
static int split_segments(int rows, int P)
{
    const int segs = (P + kSegment - 1) / kSegment;
    return P > 32768 && P <= kBitmapRow && (long)rows * segs <= (segs >= 8 ? 512 : 256) ? segs : 0;
}

size_t topk_final_scratch_bytes(int rows, int P)
{
    return (size_t)rows * split_segments(rows, P) * (2 * kBudgetBlock + kSegment) * sizeof(uint16_t) +
           (split_segments(rows, P) ? (size_t)rows * sizeof(uint4) : 0);
}

// Few enough bytes of a head's retained rows for its workgroup (whole passes, us, a launch of its own / in the
// selection: 4 heads x 64 rows of 256 bytes 34.2 / 31.9, 8 heads x 256 19.9 / 16.2 with key norms and 54.7 / 55.3 with
// two rounds, 256 heads x 256 305.5 / 302.6, 1024 x 256 1019 / 1014; 8 heads x 512 rows 44.9 / 47.9).
bool topk_final_gathers(int P, int max_budget, int row_bytes) { return P <= 32768 && (long)max_budget * row_bytes <= (64 << 10); }

hipError_t launch_topk_final(float *scores, int P, int rows, const LayerPlan &plan, int w, int32_t *idx,
                             const DecayArgs &update, const GatherArgs &gather, void *scratch, hipStream_t st)
{
    if (rows <= 0) return hipSuccess;
    if (P <= 32768) {
        switch (update.items) {
            case 0: return launch_budget_d<0>(scores, P, rows, plan, w, idx, update, gather, st);
            case 1: return launch_budget_d<1>(scores, P, rows, plan, w, idx, update, gather, st);
            case 2: return launch_budget_d<2>(scores, P, rows, plan, w, idx, update, gather, st);
            case 4: return launch_budget_d<4>(scores, P, rows, plan, w, idx, update, gather, st);
            default: return hipErrorInvalidValue;
        }
    }
    if (update.items || gather.Kout) return hipErrorInvalidValue;
    const int segs = scratch ? split_segments(rows, P) : 0;
    if (segs) {
        SplitScratch sc;
        sc.range = reinterpret_cast<uint4 *>(scratch);
        sc.above = reinterpret_cast<uint16_t *>(sc.range + rows);
        sc.order = sc.above + (size_t)rows * segs * 2 * kBudgetBlock;
        if (!allow_big_lds((const void *)split_select_kernel, 140 * 1024)) return hipGetLastError();
        // (a row's workgroups `rows` apart in both launches: with 8 rows each stays on one XCD)
        hipLaunchKernelGGL(split_count_kernel, dim3(rows, segs), dim3(kBudgetBlock), 0, st, scores, P, sc);
        hipLaunchKernelGGL(split_select_kernel, dim3(rows, segs), dim3(kBudgetBlock), (size_t)kBudgetList * 8, st, scores, P,
                           idx, P, w, sc, plan);
        return hipGetLastError();
    }
    if (P <= kBitmapRow) {
        if (!allow_big_lds((const void *)budget_select_long_kernel, 140 * 1024)) return hipGetLastError();
        const size_t words = (size_t)(P + kWave - 1) / kWave;
        hipLaunchKernelGGL(budget_select_long_kernel, dim3(rows), dim3(kBudgetBlock),
                           words * 8 + (size_t)kBudgetList * 8, st, scores, P, idx, P, w, plan);
    } else {
        hipLaunchKernelGGL((topk_rows_stream_kernel<1024, true>), dim3(rows), dim3(1024), 0, st, scores, (long)P, P,
                           0, idx, 0L, (float *)nullptr, 0L, P, w, plan);
    }
    return hipGetLastError();
}

}  // namespace gkv
