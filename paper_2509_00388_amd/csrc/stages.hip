// Pooling of the window votes, the signal-propagation update (Eq. 4 / Eq. 5)
// and the K/V gather of the retained rows.
#include "common.hpp"
#include "decay.hpp"
#include "kernels.hpp"

#include <mutex>
#include <set>
#include <utility>

namespace gkv {

bool allow_big_lds(const void *kernel, int bytes)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void *>> done;   // (device, kernel) pairs that are opted in
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count({dev, kernel})) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        return false;
    done.insert({dev, kernel});
    return true;
}

// scores[h, j] = (1/div) * sum_g pool(votes[h*Gv + g, j-half .. j+half]).
// Average pooling pads with zeros and divides by the kernel size; max pooling
// ignores positions outside the row.
__global__ __launch_bounds__(256) void pool_group_kernel(const float *__restrict__ votes, int Gv,
                                                         int P, int pool_kernel, int pool_mode,
                                                         float div, float *__restrict__ scores)
{
    const int h = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= P) return;
    const int half = (pool_kernel - 1) / 2;
    const int lo = max(0, j - half), hi = min(P - 1, j + half);
    float total = 0.f;
    for (int g = 0; g < Gv; ++g) {
        const float *v = votes + ((long)h * Gv + g) * P;
        float acc;
        if (pool_mode == 0) {
            acc = 0.f;
            for (int t = lo; t <= hi; ++t) acc += v[t];
            acc = acc / (float)pool_kernel;
        } else {
            acc = -INFINITY;
            for (int t = lo; t <= hi; ++t) acc = fmaxf(acc, v[t]);
        }
        total += acc;
    }
    scores[(long)h * P + j] = total / div;
}

// Average pooling is linear, so the Gv vote rows of a head are added first (one
// coalesced load per row and thread) and the sum is pooled once out of an LDS tile
// with a halo.  Same value as pooling each row and adding, up to fp32 rounding order.
constexpr int kPoolHalo = 16;
// kPoolTile outputs per workgroup: 2048 (8 per thread, enough loads in flight per CU) when
// there are many heads, 256 when the grid would otherwise not fill the chip.
template <int kPoolTile>
__global__ __launch_bounds__(256) void pool_avg_kernel(const float *__restrict__ votes, int Gv, int P,
                                                       int pool_kernel, float div,
                                                       float *__restrict__ scores)
{
    __shared__ float tile[kPoolTile + 2 * kPoolHalo];
    const int h = blockIdx.y, j0 = blockIdx.x * kPoolTile, tid = threadIdx.x;
    const int half = (pool_kernel - 1) / 2;
    for (int u = tid; u < kPoolTile + 2 * kPoolHalo; u += 256) {
        const int j = j0 - kPoolHalo + u;
        float v = 0.f;                               // zero padding outside the row
        if (j >= 0 && j < P && u >= kPoolHalo - half && u < kPoolTile + kPoolHalo + half)
            for (int g = 0; g < Gv; ++g) v += votes[((long)h * Gv + g) * P + j];
        tile[u] = v;
    }
    __syncthreads();
    for (int o = tid; o < kPoolTile; o += 256) {
        const int j = j0 + o;
        if (j >= P) break;
        float acc = 0.f;
        for (int t = -half; t <= half; ++t) acc += tile[kPoolHalo + o + t];
        scores[(long)h * P + j] = acc / (float)pool_kernel / div;
    }
}

// Bitonic sort of npad 64-bit keys in LDS by one workgroup of NW waves.  Wave w
// owns pairs [w*Q, (w+1)*Q), Q = npad / (2 NW).  For compare distances j <= Q those
// pairs touch only elements [2wQ, 2(w+1)Q), so such stages need no workgroup barrier:
// LDS operations of one wave complete in order.  Only the stages with j > Q
// synchronise the workgroup.
template <int NW>
__device__ __forceinline__ void bitonic_sort_lds(uint64_t *keys, int npad, int lane, int wv)
{
    const int Q = npad / (2 * NW);
    for (int k = 2; k <= npad; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const bool wide = j > Q;
            if (wide) __syncthreads();
            for (int e = wv * Q + lane; e < (wv + 1) * Q; e += kWave) {
                const int t = ((e & ~(j - 1)) << 1) | (e & (j - 1)), u = t + j;
                const uint64_t a = keys[t], b = keys[u];
                const bool up = (t & k) == 0;
                if ((a > b) == up) { keys[t] = b; keys[u] = a; }
            }
            if (wide) __syncthreads();
            else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
    }
    __syncthreads();
}

// The update as a launch of its own.
template <typename Cell, int BLOCK, int ITEMS, bool EDGES>
__global__ __launch_bounds__(BLOCK) void decay_chain_kernel(
    float *__restrict__ scores, int P, int count, int cells, const int32_t *__restrict__ nbr,
    const float *__restrict__ nbr_e, float alpha, int signal)
{
    extern __shared__ __align__(16) unsigned char chain_lds[];
    const long h = blockIdx.x;
    decay_chain<Cell, BLOCK, ITEMS, EDGES>(scores + h * P, count, cells, nbr + h * count, nbr_e + h * count, alpha,
                                           signal, chain_lds, threadIdx.x);
}

// 8192 < S*m <= 16384 and nodes beyond 2^18: the triples are sorted by (node, slot) in LDS (128 KiB of
// keys); the first triple of every node multiplies that node's factors in ascending slot order and
// writes the node's score once.  Edge weights come from global memory.
template <int NT>
__global__ __launch_bounds__(NT) void decay_sorted_kernel(
    float *__restrict__ scores, int P, int count, int npad, const int32_t *__restrict__ nbr,
    const float *__restrict__ nbr_e, float alpha, int signal)
{
    extern __shared__ uint64_t keys[];     // (node << 32) | triple id
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t *nb = nbr + (long)h * count;
    const float *ne = nbr_e + (long)h * count;
    float *s = scores + (long)h * P;
    for (int t = tid; t < npad; t += NT)
        keys[t] = t < count ? (((uint64_t)(uint32_t)nb[min(t, count - 1)] << 32) | (uint32_t)t) : ~0ull;
    __syncthreads();
    bitonic_sort_lds<NT / kWave>(keys, npad, lane, wv);
    for (int t = tid; t < count; t += NT) {
        const uint64_t key = keys[t];
        const uint32_t node = (uint32_t)(key >> 32);
        if (t > 0 && (uint32_t)(keys[t - 1] >> 32) == node) continue;   // not the first of its node
        if (signal == 2) { s[node] = -INFINITY; continue; }
        const float sj = s[node];
        float f = 1.0f;
        for (int u = t; u < count; ++u) {
            const uint64_t ku = keys[u];
            if ((uint32_t)(ku >> 32) != node) break;
            f *= signal_factor(ne[(uint32_t)ku], alpha, signal, sj < 0.f);
        }
        s[node] = sj * f;
    }
}

// The same update by a radix sort, for up to BLOCK * ITEMS triples whose (node, triple)
// pair fits 32 bits.  Key = node << kTripleBits | triple id.
// The triple ids ascend in the input, and a least-significant-digit radix sort is stable, so
// sorting by the node bits alone (6 bits a pass) leaves the triples of a node in ascending
// id, i.e. ascending source order -- Eq. 5's fixed order.  Per pass every wave ranks the keys of
// its own contiguous block: the lanes that hold the same digit find each other with six wave
// votes, the lowest of them adds their number to the wave's counter of that digit, and a
// block-wide scan of the (digit, wave) counters gives every key its place; three barriers a
// pass.  Then the first triple of every node multiplies that node's factors and writes its
// score once.  Two key buffers in LDS (8 bytes per triple in all), of which the edges take the one that is free by
// then: a thread asks for its edges up front and for all its nodes' scores at once, and the products, four factors
// at a time, wait for the LDS only.  (Edge after edge from memory, score after score: 105 us for 256 heads of 16384 triples and 131008 nodes, this way 82.)
template <int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void decay_radix_kernel(
    float *__restrict__ scores, int P, int count, int node_bits, const int32_t *__restrict__ nbr,
    const float *__restrict__ nbr_e, float alpha, int signal)
{
    constexpr int NW = BLOCK / kWave, NPAD = BLOCK * ITEMS;
    static_assert(NPAD <= (1 << kTripleBits), "triple ids must fit kTripleBits");
    extern __shared__ uint32_t radix_lds[];
    uint32_t *buf_a = radix_lds, *buf_b = radix_lds + NPAD;   // [NPAD] each
    __shared__ uint32_t cnt_s[NW][64];                        // keys of each digit in each wave's block
    __shared__ uint32_t wave_sum[NW];
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t *nb = nbr + (long)h * count;
    const float *ne = nbr_e + (long)h * count;
    float *s = scores + (long)h * P;
    const uint64_t below = (1ull << lane) - 1ull;

    // keys of this wave's block, entry it * 64 + lane of it: registers hold them through a pass
    uint32_t key[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int t = (wv * ITEMS + it) * kWave + lane;
        const uint32_t node = (uint32_t)nb[min(t, count - 1)];
        key[it] = t < count ? (node << kTripleBits) | (uint32_t)t : 0xffffffffu;   // padding sorts last
    }
    float e[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) e[it] = ne[min((wv * ITEMS + it) * kWave + lane, count - 1)];
    uint32_t *src_buf = buf_a, *dst_buf = buf_b;
    for (int shift = kTripleBits; shift < kTripleBits + node_bits; shift += 6) {
        for (int i = lane; i < 64; i += kWave) cnt_s[wv][i] = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        uint32_t place[ITEMS];   // digit << 16 | rank among the wave's keys of that digit
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const uint32_t d = (key[it] >> shift) & 63u;
            uint64_t peers = ~0ull;   // lanes whose key has the same digit
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const uint64_t v = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? v : ~v;
            }
            const int leader = __ffsll((long long)peers) - 1;
            uint32_t base = 0;
            if (lane == leader) base = atomicAdd(&cnt_s[wv][d], (uint32_t)__popcll(peers));
            base = __shfl(base, leader, kWave);
            place[it] = (d << 16) | (base + (uint32_t)__popcll(peers & below));
        }
        __syncthreads();
        // exclusive scan of the counters in (digit, wave) order: thread t <-> digit t / NW, wave t % NW
        uint32_t run = 0;
        {
            uint32_t v = 0;
            if (tid < 64 * NW) v = cnt_s[tid % NW][tid / NW];
            uint32_t incl = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(incl, o, kWave);
                if (lane >= o) incl += u;
            }
            if (lane == 63) wave_sum[wv] = incl;
            __syncthreads();
            uint32_t before = 0;
            for (int u = 0; u < wv; ++u) before += wave_sum[u];
            run = before + incl - v;
            __syncthreads();      // every counter is read before it is overwritten with its offset
            if (tid < 64 * NW) cnt_s[tid % NW][tid / NW] = run;
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            dst_buf[cnt_s[wv][place[it] >> 16] + (place[it] & 0xffffu)] = key[it];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) key[it] = dst_buf[(wv * ITEMS + it) * kWave + lane];
        uint32_t *tmp = src_buf; src_buf = dst_buf; dst_buf = tmp;
    }
    // the sorted keys sit in registers (position (wv * ITEMS + it) * 64 + lane) and in src_buf
    if (src_buf == buf_a) {   // (no pass at all: node_bits = 0 cannot happen, P >= 2; keep the buffer valid)
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) buf_a[(wv * ITEMS + it) * kWave + lane] = key[it];
        __syncthreads();
    }
    const uint32_t *sorted = src_buf;
    constexpr uint32_t kTriple = (1u << kTripleBits) - 1u;
    float *edge = reinterpret_cast<float *>(dst_buf);   // (read into registers before the pass's last barrier)
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) edge[(wv * ITEMS + it) * kWave + lane] = e[it];
    // the first triples of their nodes, and those nodes' scores
    bool first[ITEMS];
    float sj[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int pos = (wv * ITEMS + it) * kWave + lane;
        const uint32_t before = pos > 0 ? sorted[pos - 1] : ~key[it];
        first[it] = pos < count && (before >> kTripleBits) != (key[it] >> kTripleBits);
        sj[it] = 0.f;
        if (first[it]) sj[it] = s[key[it] >> kTripleBits];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int pos = (wv * ITEMS + it) * kWave + lane;
        if (!first[it]) continue;
        const uint32_t node = key[it] >> kTripleBits;
        if (signal == 2) { s[node] = -INFINITY; continue; }
        const bool neg = sj[it] < 0.f;
        float f = signal_factor(edge[key[it] & kTriple], alpha, signal, neg);
        for (int u = pos + 1; u < count; u += 4) {
            uint32_t ku[4];
            float eu[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) ku[k] = sorted[min(u + k, count - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k) eu[k] = edge[ku[k] & kTriple];
            bool same = true;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                same = same && u + k < count && (ku[k] >> kTripleBits) == node;
                f = same ? f * signal_factor(eu[k], alpha, signal, neg) : f;
            }
            if (!same) break;
        }
        s[node] = sj[it] * f;
    }
}

// Same update without the sort, for S*m beyond the LDS capacity: sources are
// applied one after the other; inside one source the m neighbours are distinct
// nodes, so they can be updated in parallel.  Multiplying s_j by the factors one
// at a time differs from multiplying by their product only in rounding order, so
// here too the product is formed first, per node, by the lowest slot that holds it.
__global__ __launch_bounds__(1024) void decay_sequential_kernel(
    float *__restrict__ scores, int P, int S, int m, const int32_t *__restrict__ nbr,
    const float *__restrict__ nbr_e, float alpha, int signal)
{
    const int h = blockIdx.x;
    const int32_t *nb = nbr + (long)h * S * m;
    const float *ne = nbr_e + (long)h * S * m;
    float *s = scores + (long)h * P;
    // Thread (a, u) owns node j = nb[a][u] if no earlier slot a' < a lists j.
    // Neighbour lists are ascending, so membership is a binary search.
    for (long t = threadIdx.x; t < (long)S * m; t += 1024) {
        const int a = (int)(t / m);
        const int32_t j = nb[t];
        bool first = true;
        for (int b = 0; b < a && first; ++b) {
            int lo = 0, hi = m - 1;
            while (lo <= hi) {
                const int mid = (lo + hi) >> 1;
                const int32_t v = nb[(long)b * m + mid];
                if (v == j) { first = false; break; }
                if (v < j) lo = mid + 1; else hi = mid - 1;
            }
        }
        if (!first) continue;
        if (signal == 2) { s[j] = -INFINITY; continue; }
        const float sj = s[j];
        const bool neg = sj < 0.f;
        float f = signal_factor(ne[t], alpha, signal, neg);
        for (int b = a + 1; b < S; ++b) {
            int lo = 0, hi = m - 1;
            while (lo <= hi) {
                const int mid = (lo + hi) >> 1;
                const int32_t v = nb[(long)b * m + mid];
                if (v == j) { f *= signal_factor(ne[(long)b * m + mid], alpha, signal, neg); break; }
                if (v < j) lo = mid + 1; else hi = mid - 1;
            }
        }
        s[j] = sj * f;
    }
}

// Kout[q, t, :] = Kc[q, idx[q, t], :] for head q = l * H + h of a batch, same for V;
// 16 bytes per thread, rows of 16 * vec_per_row bytes.  Outputs and idx are packed
// layer after layer (layer l holds H * B_l rows).
template <bool ONCE>
__global__ __launch_bounds__(256) void gather_kernel(const u32x4 *__restrict__ Kc,
                                                     const u32x4 *__restrict__ Vc,
                                                     const int32_t *__restrict__ idx, int N,
                                                     int vec_per_row, u32x4 *__restrict__ Kout,
                                                     u32x4 *__restrict__ Vout, LayerPlan plan)
{
    const int q = blockIdx.y;
    const int l = q / plan.heads_per_layer, hl = q % plan.heads_per_layer;
    const int B = plan.budget[l];
    const long g = (long)blockIdx.x * 256 + threadIdx.x;
    if (g >= (long)B * vec_per_row) return;
    const int t = (int)(g / vec_per_row), c = (int)(g % vec_per_row);
    const long out_row = plan.row_off[l] + (long)hl * B + t;
    const int32_t j = idx[out_row];
    const long src = ((long)q * N + j) * vec_per_row + c;
    const long dst = out_row * vec_per_row + c;
    const u32x4 *in = blockIdx.z == 0 ? Kc : Vc;
    u32x4 *out = blockIdx.z == 0 ? Kout : Vout;
    if (ONCE) __builtin_nontemporal_store(in[src], out + dst);
    else out[dst] = in[src];
}

template <typename T>
__global__ __launch_bounds__(256) void copy_kernel(const T *__restrict__ src, T *__restrict__ dst,
                                                   long n)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_pool_group(const float *votes, int Hkv, int Gv, int P, int pool_kernel,
                             int pool_mode, float div, float *scores, hipStream_t st)
{
    if (pool_mode == 0 && pool_kernel <= 2 * kPoolHalo + 1) {
        if ((long)((P + 2047) / 2048) * Hkv >= 1024)
            hipLaunchKernelGGL(pool_avg_kernel<2048>, dim3((P + 2047) / 2048, Hkv), dim3(256), 0, st, votes,
                               Gv, P, pool_kernel, div, scores);
        else
            hipLaunchKernelGGL(pool_avg_kernel<256>, dim3((P + 255) / 256, Hkv), dim3(256), 0, st, votes,
                               Gv, P, pool_kernel, div, scores);
    } else {
        hipLaunchKernelGGL(pool_group_kernel, dim3((P + 255) / 256, Hkv), dim3(256), 0, st, votes, Gv,
                           P, pool_kernel, pool_mode, div, scores);
    }
    return hipGetLastError();
}

template <typename Cell, int BLOCK, int ITEMS, bool EDGES>
static hipError_t launch_decay_chain(float *scores, int Hkv, int P, int count, const int32_t *nbr,
                                     const float *nbr_e, float alpha, int signal, hipStream_t st)
{
    const int slots = BLOCK * ITEMS;
    const int cells = decay_chain_cells(slots);
    const size_t lds = decay_chain_lds<Cell>(cells, slots, EDGES);
    if (lds > 65536 && !allow_big_lds((const void *)decay_chain_kernel<Cell, BLOCK, ITEMS, EDGES>))
        return hipGetLastError();
    hipLaunchKernelGGL((decay_chain_kernel<Cell, BLOCK, ITEMS, EDGES>), dim3(Hkv), dim3(BLOCK), lds, st, scores, P,
                       count, cells, nbr, nbr_e, alpha, signal);
    return hipGetLastError();
}

// Triples per thread (1, 2 or 4) of an update that the next kernel over the same rows can take along, 0 if
// it needs a launch of its own: up to 4096 triples, rows that kernel keeps in registers.
int decay_rides_along(int P, int S, int m)
{
    const long count = (long)S * m;
    if (P > 32768 || count > 4096) return 0;
    return count <= 1024 ? 1 : (count <= 2048 ? 2 : 4);
}

hipError_t launch_decay(float *scores, int Hkv, int P, int S, int m, const int32_t *nbr,
                        const float *nbr_e, float alpha, int signal, hipStream_t st)
{
    const long count = (long)S * m;
    const bool narrow = P < (1 << (32 - kTripleBits));   // node and triple id share 32 bits (all ones is a free cell)
#define GKV_DECAY(CELL, BLOCK, ITEMS, EDGES) \
    return launch_decay_chain<CELL, BLOCK, ITEMS, EDGES>(scores, Hkv, P, (int)count, nbr, nbr_e, alpha, signal, st)
    if (narrow) {
        // Many triples in many long rows: the chains' scattered score reads queue up and the sort,
        // which reads a node's score once, wins (us, sort / chains: 256 heads of 32736 nodes with 8192
        // triples 45 / 52, with 16384 87 / 106; 64 heads of 131040 nodes 46 / 55 and 75 / 92).  With few
        // heads or short rows the chains do (8 heads of 32736 nodes 32 / 28 and 60 / 45; 256 heads of 8160
        // nodes 48 / 22 and 139 / 46), and up to 4096 triples always (256 heads of 32736 nodes 30 / 25).
        if (count > 4096 && count <= 16384 && P > 16384 && Hkv >= 32) {
            int node_bits = 1;
            while ((1L << node_bits) < P) ++node_bits;
            if (!allow_big_lds((const void *)decay_radix_kernel<1024, 16>, 16384 * 8)) return hipGetLastError();
            if (count <= 8192)
                hipLaunchKernelGGL((decay_radix_kernel<1024, 8>), dim3(Hkv), dim3(1024), (size_t)8192 * 8, st, scores, P,
                                   (int)count, node_bits, nbr, nbr_e, alpha, signal);
            else
                hipLaunchKernelGGL((decay_radix_kernel<1024, 16>), dim3(Hkv), dim3(1024), (size_t)16384 * 8, st, scores, P,
                                   (int)count, node_bits, nbr, nbr_e, alpha, signal);
            return hipGetLastError();
        }
        if (count <= 256) GKV_DECAY(uint32_t, 256, 1, true);
        if (count <= 1024) GKV_DECAY(uint32_t, 1024, 1, true);
        if (count <= 2048) GKV_DECAY(uint32_t, 1024, 2, true);
        if (count <= 4096) GKV_DECAY(uint32_t, 1024, 4, true);
        if (count <= 8192) GKV_DECAY(uint32_t, 1024, 8, true);
        if (count <= 16384) GKV_DECAY(uint32_t, 1024, 16, false);   // (its edges would not fit beside the cells)
    } else {
        if (count <= 4096) GKV_DECAY(uint64_t, 1024, 4, true);
        if (count <= 8192) GKV_DECAY(uint64_t, 1024, 8, true);
        if (count <= 16384) {
            // 16 waves sort the 16384 keys of 128 KiB of dynamic LDS
            if (!allow_big_lds((const void *)decay_sorted_kernel<1024>, 16384 * 8)) return hipGetLastError();
            hipLaunchKernelGGL(decay_sorted_kernel<1024>, dim3(Hkv), dim3(1024), (size_t)16384 * 8, st, scores, P,
                               (int)count, 16384, nbr, nbr_e, alpha, signal);
            return hipGetLastError();
        }
    }
#undef GKV_DECAY
    hipLaunchKernelGGL(decay_sequential_kernel, dim3(Hkv), dim3(1024), 0, st, scores, P, S, m, nbr, nbr_e, alpha,
                       signal);
    return hipGetLastError();
}

hipError_t launch_gather(const void *Kc, const void *Vc, const int32_t *idx, int heads, int N,
                         const LayerPlan &plan, int max_budget, int row_bytes, void *Kout, void *Vout,
                         hipStream_t st)
{
    const int vpr = row_bytes / 16;
    const long per_head = (long)max_budget * vpr;
    const bool once = reads_past_caches((size_t)heads * N * row_bytes);
    hipLaunchKernelGGL(once ? gather_kernel<true> : gather_kernel<false>, dim3((unsigned)((per_head + 255) / 256), heads, 2),
                       dim3(256), 0, st, (const u32x4 *)Kc, (const u32x4 *)Vc, idx, N, vpr, (u32x4 *)Kout, (u32x4 *)Vout, plan);
    return hipGetLastError();
}

hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel<int32_t>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       src, dst, n);
    return hipGetLastError();
}

hipError_t launch_copy_f32(const float *src, float *dst, long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel<float>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src,
                       dst, n);
    return hipGetLastError();
}

}  // namespace gkv
