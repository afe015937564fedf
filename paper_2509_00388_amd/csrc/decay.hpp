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
            const bool neg = sj[b] < 0.f;
            float f = 1.0f;
            if (next[t] == kChainEnd) {
                f *= signal_factor(e[b], alpha, signal, neg);
            } else {
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
                    for (int i = 0; i < kLinks; ++i) {
                        const uint32_t u = min(low[i], (uint32_t)count - 1u);
                        el[i] = EDGES ? edge[u] : ne[u];
                    }
#pragma unroll
                    for (int i = 0; i < kLinks; ++i)
                        if (low[i] != kChainEnd) f *= signal_factor(el[i], alpha, signal, neg);
                    last = low[kLinks - 1];
                    from = last + 1;
                }
            }
            s[node[q]] = sj[b] * f;
        }
    }
}

}  // namespace gkv
