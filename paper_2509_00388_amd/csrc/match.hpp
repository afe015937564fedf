// From the second round on: where each source gets its neighbour list from.
#pragma once
#include "common.hpp"
#include "decay.hpp"
#include "kernels.hpp"

namespace gkv {

constexpr int kMatchBlock = 1024;

// Where each source of this round (cur [S], ascending) of head h gets its neighbour list from:
//   - it was a source in the previous round (prev, ascending): its list (prev_nbr, prev_e
//     [Hkv, S, m]) is copied to its slot of this round (nbr, nbr_e);
//   - it is one of the head's speculative rows (entries S .. S + X of ext [Hkv, S + X],
//     ascending, whose candidate lists the first round's filter pass built in rows
//     S .. of the per-row buffers) and
//     those lists are complete (the head raised no overflow flag in the first round): the
//     exact select runs on that row;
//   - otherwise it goes, in order, to new_src[h, 0 .. n_new[h]) for another bound and filter
//     pass, which uses rows 0 .. of the per-row buffers (the candidates of the first round's
//     sources are no longer needed once their lists are selected).
// The selections to run are listed as (candidate row, source slot) in sel_row / sel_pos
// [Hkv, S], n_sel[h] of them.  spec_bad [Hkv] remembers across rounds whether a head's
// speculative lists may be used: the first match of a call sets it from the overflow flags
// of the first round (first != 0), later ones read it.  One workgroup of kMatchBlock threads per
// head; lds holds 2 S + X words.  match_load() fetches the lists the sources are looked up in; it goes
// in front of whatever finds the sources, so that its loads are back by then.  Returns whether the
// head's speculative lists are of no use.
__device__ __forceinline__ bool match_load(const MatchArgs &a, int h, int32_t *lds, int tid)
{
    const int S = a.S, X = a.X;
    for (int b = tid; b < S; b += kMatchBlock) lds[b] = a.prev_src[(long)h * S + b];
    for (int b = tid; b < X; b += kMatchBlock) lds[2 * S + b] = a.ext[(long)h * (S + X) + S + b];   // behind the S sources
    bool bad = X == 0;
    if (X > 0) {
        bad = a.first ? a.overflow[h] != 0 : a.spec_bad[h] != 0;
        if (a.first && tid == 0) a.spec_bad[h] = bad ? 1 : 0;
    }
    return bad;
}

// The lists that stay are copied: the neighbourhood of a source does not depend on the scores.  Lists that the
// thread holds already (the triples of the update that rode along: entry q * kMatchBlock + tid of the previous
// round's lists) are not read again.
template <int D>
__device__ __forceinline__ void match_copy(const MatchArgs &a, int h, const int32_t *code_s, const int32_t *to_s,
                                           const Triples<D> &tri, int tid)
{
    const long row0 = (long)h * a.S;
    const int entries = a.S * a.m;   // (lists are kept for S <= 4096 and m <= 1024)
    if constexpr (D > 0) {
#pragma unroll
        for (int q = 0; q < D; ++q) {
            const int u = q * kMatchBlock + tid, s = min(u, entries - 1) / a.m, to = to_s[s];
            if (u < entries && to >= 0) {
                a.nbr[(row0 + to) * a.m + (u - s * a.m)] = (int32_t)tri.node[q];
                a.nbr_e[(row0 + to) * a.m + (u - s * a.m)] = tri.e[q];
            }
        }
        return;
    }
    for (int u0 = tid; u0 < entries; u0 += 4 * kMatchBlock) {
        int32_t n[4];
        float e[4];
        bool kept[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {   // (loads of four entries leave together)
            const int u = min(u0 + v * kMatchBlock, entries - 1), s = u / a.m;
            const int from = code_s[s];
            const long at = (row0 + max(from, 0)) * a.m + (u - s * a.m);
            kept[v] = u0 + v * kMatchBlock < entries && from >= 0;
            n[v] = a.prev_nbr[at];
            e[v] = a.prev_e[at];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (kept[v]) {
                a.nbr[row0 * a.m + u0 + v * kMatchBlock] = n[v];
                a.nbr_e[row0 * a.m + u0 + v * kMatchBlock] = e[v];
            }
    }
}

// (A barrier lies between match_load() and this; to_s [S] is set to -1 in front of it if D > 0.)
template <int D>
__device__ __forceinline__ void match_head(const MatchArgs &a, int h, bool bad, const int32_t *cur, int32_t *lds,
                                           int32_t *to_s, int32_t *wave_new, int32_t *wave_fb, const Triples<D> &tri,
                                           int tid)
{
    constexpr int NW = kMatchBlock / kWave;
    const int S = a.S, X = a.X, lane = tid & 63, wv = tid >> 6;
    int32_t *prev_s = lds, *code_s = lds + S, *spec_s = lds + 2 * S;
    const long row0 = (long)h * S;
    // first slot of a sorted list that holds i or more
    auto lower_bound = [](const int32_t *list, int n, int32_t i) {
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (list[mid] < i) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    int base = 0, base_fb = 0;
    for (int s0 = 0; s0 < S; s0 += kMatchBlock) {
        const int s = s0 + tid;
        int i = 0, found = -1, spec_at = -1;
        if (s < S) {
            i = cur[s];
            const int lo = lower_bound(prev_s, S, i);
            if (lo < S && prev_s[lo] == i) found = lo;
            if (found < 0 && !bad) {
                const int u = lower_bound(spec_s, X, i);
                if (u < X && spec_s[u] == i) spec_at = u;
            }
        }
        const bool is_new = s < S && found < 0, is_fb = is_new && spec_at < 0;
        const uint64_t mask = __ballot(is_new), mask_fb = __ballot(is_fb);
        if (lane == 0) { wave_new[wv] = (int32_t)__popcll(mask); wave_fb[wv] = (int32_t)__popcll(mask_fb); }
        __syncthreads();
        int before = base, total = 0, before_fb = base_fb, total_fb = 0;
        for (int u = 0; u < NW; ++u) {
            if (u < wv) { before += wave_new[u]; before_fb += wave_fb[u]; }
            total += wave_new[u];
            total_fb += wave_fb[u];
        }
        if (s < S) code_s[s] = found;
        if (D > 0 && found >= 0) to_s[found] = s;
        if (is_new) {
            const int x = before + (int)votes_below(mask);
            int crow = S + spec_at;
            if (is_fb) {
                const int r = before_fb + (int)votes_below(mask_fb);
                a.new_src[row0 + r] = i;
                crow = r;
            }
            a.sel_row[row0 + x] = crow;
            a.sel_pos[row0 + x] = s;
        }
        base += total;
        base_fb += total_fb;
        __syncthreads();
    }
    if (tid == 0) {
        a.n_new[h] = base_fb;
        a.n_sel[h] = base;
    }
    match_copy<D>(a, h, code_s, to_s, tri, tid);
}

}  // namespace gkv
