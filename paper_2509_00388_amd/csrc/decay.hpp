// Eq. 5's update of one head by one workgroup, as a launch of its own (stages.hip) or in front of a kernel
// that takes a head's scores per workgroup too (select.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace gkv {

// Factor of one edge (Eq. 4 / Eq. 5).  The signal acts on the magnitude of the score the
// round started with: the decay takes alpha * e * |s| away, the enhanced signal adds it, so
// for a negative score (an indicator such as minus the key norm) the signs swap and the
// decay still lowers the score.  For s >= 0 this is (1 - alpha e) as printed.
__device__ __forceinline__ float signal_factor(float e, float alpha, int signal, bool negative)
{
    return ((signal == 1) != negative) ? fmaf(alpha, e, 1.0f) : fmaf(-alpha, e, 1.0f);
}

// Eq. 5 for one round, S*m <= 16384.  One workgroup per head, no sort and no float atomics.  Every
// (source slot, node, edge) triple t finds its node's cell in an LDS hash table (open addressing; an
// integer compare-and-swap claims a cell), and the triples of a node form a chain: the cell holds
// the last one that came, next[] the one before it.  The thread whose triple ends up at the head of
// a chain multiplies the chain's factors in ascending t -- sources are stored in ascending index
// order, so the product is Eq. 5's with a fixed floating-point order whatever the order the chain
// was built in -- and writes the node's score once.  Most chains have one link; a longer one is
// walked once per kLinks links.  What bounds it is latency: three dependent loads and one LDS round trip.
// (A radix sort of the triples: 12.5 us for 8 heads of 2048 triples, 19 us for 256; this way 7.7 and
// 13 us.)
// Cell: node and triple in one word, 32 bits (node < 2^18) or 64.
constexpr int kTripleBits = 14;   // triple ids below 16384
constexpr uint32_t kChainEnd = 0xffffu;
constexpr int kLinks = 8;         // triples of a chain that one walk puts in order

template <typename Cell> struct CellOf;
template <> struct CellOf<uint32_t> {
    static constexpr int kShift = kTripleBits;
    __device__ static __forceinline__ uint32_t swap_if_free(uint32_t *c, uint32_t v) { return atomicCAS(c, ~0u, v); }
    __device__ static __forceinline__ uint32_t exchange(uint32_t *c, uint32_t v) { return atomicExch(c, v); }
};
template <> struct CellOf<uint64_t> {
    static constexpr int kShift = 32;
    __device__ static __forceinline__ uint64_t swap_if_free(uint64_t *c, uint64_t v)
    {
        return atomicCAS(reinterpret_cast<unsigned long long *>(c), ~0ull, (unsigned long long)v);
    }
    __device__ static __forceinline__ uint64_t exchange(uint64_t *c, uint64_t v)
    {
        return atomicExch(reinterpret_cast<unsigned long long *>(c), (unsigned long long)v);
    }
};

// Product of the factors of the chain that ends with triple t (edge e), in ascending triples; edge_of(u) = edge of
// triple u, whatever lies beyond the last one for any other u.
template <typename EdgeOf>
__device__ __forceinline__ float chain_factor(int t, float e, const uint16_t *next, bool neg, float alpha, int signal,
                                              EdgeOf &&edge_of)
{
    float f = 1.0f;
    if (next[t] == kChainEnd) {
        f *= signal_factor(e, alpha, signal, neg);
        return f;
    }
    // the chain's triples in ascending order, the next kLinks of them by each walk
    for (uint32_t from = 0, last = 0; last != kChainEnd;) {
        uint32_t low[kLinks];
#pragma unroll
        for (int i = 0; i < kLinks; ++i) low[i] = kChainEnd;
        for (uint32_t u = (uint32_t)t; u != kChainEnd; u = next[u]) {
            uint32_t x = u >= from ? u : kChainEnd;
#pragma unroll
            for (int i = 0; i < kLinks; ++i) {
                const uint32_t keep = min(low[i], x);
                x = max(low[i], x);
                low[i] = keep;
            }
        }
        float el[kLinks];
#pragma unroll
        for (int i = 0; i < kLinks; ++i) el[i] = edge_of(low[i]);
#pragma unroll
        for (int i = 0; i < kLinks; ++i)
            if (low[i] != kChainEnd) f *= signal_factor(el[i], alpha, signal, neg);
        last = low[kLinks - 1];
        from = last + 1;
    }
    return f;
}

// Bytes of dynamic LDS: cells, edges (unless they stay in global memory), links.
template <typename Cell> size_t decay_chain_lds(int cells, int slots, bool edges)
{
    return (size_t)cells * sizeof(Cell) + (size_t)slots * (edges ? 4 : 0) + (size_t)slots * 2;
}
// Cells for so many slots: twice as many, beyond 8192 one and a half times (LDS holds no more).
inline int decay_chain_cells(int slots) { return slots < 8192 ? 2 * slots : slots + slots / 2; }

// s: the head's scores; nb, ne: its triples; decay_lds: decay_chain_lds() bytes.  The caller puts a
// barrier behind it before it reads the scores.
template <typename Cell, int BLOCK, int ITEMS, bool EDGES>
__device__ __forceinline__ void decay_chain(float *s, int count, int cells, const int32_t *nb, const float *ne,
                                            float alpha, int signal, unsigned char *decay_lds, int tid)
{
    // Few triples: every thread asks for its nodes' scores at once, behind the node numbers.  Many:
    // only the heads of chains do, at the end, four at a time -- a score read is a 64-byte line for
    // four bytes, and with 16384 triples about half the nodes occur more than once.
    constexpr bool kEarly = ITEMS <= 4;
    constexpr int SLOTS = BLOCK * ITEMS, SH = CellOf<Cell>::kShift, B = kEarly ? ITEMS : 4;
    constexpr Cell kFree = ~(Cell)0;
    Cell *cell = reinterpret_cast<Cell *>(decay_lds);                     // [cells]
    float *edge = reinterpret_cast<float *>(cell + cells);                // [SLOTS] if EDGES
    uint16_t *next = reinterpret_cast<uint16_t *>(edge + (EDGES ? SLOTS : 0));
    // (unconditional, clamped loads: those of a batch leave together)
    uint32_t node[ITEMS], at[ITEMS];
    float early[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) node[q] = (uint32_t)nb[min(q * BLOCK + tid, count - 1)];
    if (EDGES) {
        float e[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) e[q] = ne[min(q * BLOCK + tid, count - 1)];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) edge[q * BLOCK + tid] = e[q];
    }
    for (int i = tid; i < cells; i += BLOCK) cell[i] = kFree;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) early[q] = kEarly ? s[node[q]] : 0.f;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int t = q * BLOCK + tid;
        at[q] = 0;
        if (t < count) {
            const Cell mine = ((Cell)node[q] << SH) | (Cell)t;
            uint32_t c = (uint32_t)(((uint64_t)(node[q] * 2654435761u) * (uint32_t)cells) >> 32);
            uint32_t link = kChainEnd;
            while (true) {   // (there are more cells than triples)
                const Cell prev = CellOf<Cell>::swap_if_free(&cell[c], mine);
                if (prev == kFree) break;
                if ((uint32_t)(prev >> SH) == node[q]) {   // the node's cell: a cell never changes its node
                    link = (uint32_t)(CellOf<Cell>::exchange(&cell[c], mine) & (((Cell)1 << kTripleBits) - 1));
                    break;
                }
                c = c + 1 < (uint32_t)cells ? c + 1 : 0u;
            }
            next[t] = (uint16_t)link;
            at[q] = c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q0 = 0; q0 < ITEMS; q0 += B) {
        bool head[B];
        float sj[B], e[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int q = q0 + b, t = q * BLOCK + tid;
            head[b] = t < count && cell[at[q]] == (((Cell)node[q] << SH) | (Cell)t);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int q = q0 + b, t = q * BLOCK + tid;
            sj[b] = kEarly ? early[q] : s[head[b] ? node[q] : 0u];
            e[b] = EDGES ? edge[t] : ne[head[b] ? t : 0];
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int q = q0 + b, t = q * BLOCK + tid;
            if (!head[b]) continue;
            if (signal == 2) { s[node[q]] = -INFINITY; continue; }
            const float f = chain_factor(t, e[b], next, sj[b] < 0.f, alpha, signal, [&](uint32_t u) {
                const uint32_t in = min(u, (uint32_t)count - 1u);
                return EDGES ? edge[in] : ne[in];
            });
            s[node[q]] = sj[b] * f;
        }
    }
}

// The same update in front of a kernel that holds the head's row in registers, entry i of thread tid being node
// i * 1024 + tid: D triples per thread, P <= 1024 ITEMS <= 32768.  A table in LDS with a word per node takes the
// place of the hash table (only the words of the triples' nodes are ever set), so a link is one exchange; the new
// scores go to memory and, through the table, into the registers that hold the old ones.  Returns with a barrier,
// behind which `mem` is free.  (Hash chains, then a read of the row: the row was ready 7.6 us into a workgroup with
// 32736 nodes and 2048 triples, 5.6 with 16384; this way 4.8 and 4.5, of which the row's own 128 KiB take 2.)
constexpr int kUpdateBlock = 1024;
// Table, marks, links and, where that fits, edges: not with four triples a thread and 32 entries, whose edges stay in
// memory.
template <int ITEMS, int D> constexpr bool update_row_edges() { return ITEMS < 32 || D < 4; }
template <int ITEMS, int D> constexpr size_t update_row_lds()
{
    return D ? (size_t)kUpdateBlock * (4 * ITEMS + 4 + (update_row_edges<ITEMS, D>() ? 4 * D : 0) + 2 * D) : 0;
}

// The thread's triples; asked for in front of the row, which takes longer.
template <int D> struct Triples {
    uint32_t node[D > 0 ? D : 1];   // node and edge of triple q * kUpdateBlock + tid
    float e[D > 0 ? D : 1];
    __device__ __forceinline__ void load(const DecayArgs &u, int h, int tid)   // (unconditional, clamped)
    {
#pragma unroll
        for (int q = 0; q < D; ++q) node[q] = (uint32_t)u.nbr[(long)h * u.count + min(q * kUpdateBlock + tid, u.count - 1)];
#pragma unroll
        for (int q = 0; q < D; ++q) e[q] = u.nbr_e[(long)h * u.count + min(q * kUpdateBlock + tid, u.count - 1)];
    }
};

template <int ITEMS, int D>
__device__ __forceinline__ void update_row(float (&val)[ITEMS], const Triples<D> &tri, float *xr, int h, const DecayArgs &u,
                                           unsigned char *mem, int tid)
{
    constexpr int BLOCK = kUpdateBlock;
    constexpr bool EDGES = update_row_edges<ITEMS, D>();
    static_assert(ITEMS <= 32, "one mark per entry of a thread");
    uint32_t *cell = reinterpret_cast<uint32_t *>(mem);                 // [BLOCK * ITEMS] by node
    uint32_t *mark = cell + BLOCK * ITEMS;                              // [BLOCK] bit i: entry i of the thread is new
    float *edge = reinterpret_cast<float *>(mark + BLOCK);              // [BLOCK * D] if EDGES
    uint16_t *next = reinterpret_cast<uint16_t *>(edge + (EDGES ? BLOCK * D : 0));
    const float *ne = u.nbr_e + (long)h * u.count;
    const uint32_t (&node)[D] = tri.node;
    const float (&e)[D] = tri.e;
    uint32_t link[D];
    float sj[D];
    bool head[D];
    mark[tid] = 0;
#pragma unroll
    for (int q = 0; q < D; ++q) cell[node[q]] = kChainEnd;   // (clamped triples set their last one's again)
#pragma unroll
    for (int q = 0; q < D; ++q) sj[q] = xr[node[q]];
    if (EDGES) {
#pragma unroll
        for (int q = 0; q < D; ++q) edge[q * BLOCK + tid] = e[q];
    }
    __syncthreads();
    // (The chains end, and are multiplied out, at the thread that links last.  All threads' first triples go first, then
    // the second ones and so on: the ends of long chains are then one to a thread and not several, one behind another.
    // 152 nodes with 20 factors each, update and selection: 45 us without the barriers, 31 with them.)
#pragma unroll
    for (int q = 0; q < D; ++q) {
        if (q > 0) __syncthreads();
        link[q] = q * BLOCK + tid < u.count ? atomicExch(&cell[node[q]], (uint32_t)(q * BLOCK + tid)) : kChainEnd;
    }
#pragma unroll
    for (int q = 0; q < D; ++q) next[q * BLOCK + tid] = (uint16_t)link[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < D; ++q) head[q] = q * BLOCK + tid < u.count && cell[node[q]] == (uint32_t)(q * BLOCK + tid);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < D; ++q) {
        if (!head[q]) continue;
        float now = -INFINITY;
        if (u.signal != 2)
            now = sj[q] * chain_factor(q * BLOCK + tid, e[q], next, sj[q] < 0.f, u.alpha, u.signal, [&](uint32_t t) {
                      const uint32_t in = min(t, (uint32_t)u.count - 1u);
                      return EDGES ? edge[in] : ne[in];
                  });
        xr[node[q]] = now;
        cell[node[q]] = __float_as_uint(now);
        atomicOr(&mark[node[q] & (BLOCK - 1)], 1u << (node[q] / BLOCK));
    }
    __syncthreads();
    const uint32_t fresh = mark[tid];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const float now = __uint_as_float(cell[i * BLOCK + tid]);
        val[i] = (fresh >> i) & 1u ? now : val[i];
    }
    __syncthreads();
}

}  // namespace gkv
