// Stage I on the matrix cores (bf16 inputs, d = 128, fp32 accumulation).
//
// Per KV head the window queries of its G query heads are stacked into one
// R x 128 operand (R = G*w rows), held in registers for the whole kernel.
// Keys stream from HBM in tiles of 128 rows through LDS (mfma_tile.hpp); each of
// the 4 key streams of a workgroup multiplies 32 of those rows, so one key block
// costs R/32 x 8 v_mfma_f32_32x32x16_bf16 and every key is read from HBM exactly
// once per pass.  256 query rows (long windows) take tiles of 64 keys instead: two key
// streams and four row groups of 64 rows in the same 8 waves, so that those keys are
// streamed once too.
//
// The column sums of a row softmax need the row statistics first, so there are
// two passes over the keys:
//   pass A  per-row running max and sum of exp over the visible keys (online,
//           kept per lane; queries are the MFMA's column dimension so that one
//           lane owns one query and no cross-lane traffic is needed);
//   pass B  logits recomputed; exp2(l*c - (max + log2 sum)) summed down the
//           query rows (queries are the MFMA's row dimension here, so the sum
//           is in-lane) and written as the vote of the key.
// Everything is done in the base-2 domain: c = scale * log2(e).
#include "common.hpp"
#include "kernels.hpp"
#include "mfma_tile.hpp"


namespace gkv {

namespace {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// (m1, z1) <- softmax-statistics merge with (m2, z2), base 2.
__device__ __forceinline__ void merge_stats(float &m1, float &z1, float m2, float z2)
{
    const float mn = fmaxf(m1, m2);
    if (mn == -INFINITY) { m1 = mn; z1 = 0.f; return; }
    z1 = z1 * fast_exp2(m1 - mn) + z2 * fast_exp2(m2 - mn);
    m1 = mn;
}

// The R query rows are split over SPLIT waves per key stream: a workgroup has 4
// key streams (wave & 3) and SPLIT row groups (wave >> 2), i.e. 4*SPLIT waves.  The
// waves of one stream load the same key block (the second load hits L1) and each
// handles NB/SPLIT of the 32-row query blocks.  With SPLIT = 2 a wave needs under
// 256 registers, two waves share a SIMD, and one wave's exp2 work overlaps the
// other's MFMAs.

// ---------------------------------------------------------------- pass A ---
// MANY: a workgroup takes `per_wg` consecutive chunks (whole tiles each) and keeps their statistics apart, so
// that a batch cuts a head's keys as a single layer does and adds the same terms in the same order.  At a
// chunk's last tile the waves park their statistics in LDS and start over; they are stored during the next
// tile, behind its barrier, while the one after that parks in the other half of the LDS.
template <int NB, int SPLIT, int STREAMS, bool MANY, bool ONCE>
__global__ __launch_bounds__(64 * STREAMS * SPLIT) void score_stats_kernel(
    const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ Qw, int N, int P, int w,
    int chunk_keys, int nchunks, int per_wg, float c, float *__restrict__ part, int R_total, int R_real, int row_base)
{
    constexpr int R = NB * kBlk, NBW = NB / SPLIT, NT = 64 * STREAMS * SPLIT, TK = kBlk * STREAMS;
    extern __shared__ __align__(16) unsigned char kt[];   // two key tiles
    __shared__ float sm[MANY ? 2 : 1][STREAMS][R], sz[MANY ? 2 : 1][STREAMS][R];
    const int h = blockIdx.y, chunk0 = blockIdx.x * (MANY ? per_wg : 1);   // the workgroup's first chunk
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv % STREAMS, row0 = (wv / STREAMS) * NBW * kBlk;   // first query row of this wave

    // (rows of the last block beyond R_real repeat the last row: their statistics go nowhere and their votes are zero)
    bf16x8 q[NBW][kSteps];
    const uint16_t *Qh = Qw + (long)h * R_real * kD;
    auto queries = [&] {
        spread_rows<NT, R, 2 * TK>(kt, tid, row0, [&](int x) { return Qh + (long)min(row_base + x, R_real - 1) * kD; }, q, [] {});
    };
    int last_vis[NBW];   // last key the lane's query of block b may see (causal window)
    float m[NBW], z[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
        last_vis[b] = P + (row_base + row0 + kBlk * b + l32) % w;
        m[b] = -INFINITY;
        z[b] = 0.f;
    }

    const uint16_t *Kh = Kc + (long)h * N * kD;
    const int k0 = chunk0 * chunk_keys, k1 = min(N, k0 + (MANY ? per_wg : 1) * chunk_keys);
    const int ntile = (k1 - k0 + TK - 1) / TK;

    // the lane's statistics -> LDS: the two half-waves (same query, other key rows) merged, one entry per stream
    auto park = [&](int half) {
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
            const float m2 = __shfl_xor(m[b], 32, kWave), z2 = __shfl_xor(z[b], 32, kWave);
            merge_stats(m[b], z[b], m2, z2);
            if (hh == 0) {
                sm[half][stream][row0 + kBlk * b + l32] = m[b];
                sz[half][stream][row0 + kBlk * b + l32] = z[b];
            }
        }
    };
    auto store = [&](int at, int half) {   // the streams' entries merged -> the statistics of chunk0 + at
        if (tid < R) {
            float mm = sm[half][0][tid], zz = sz[half][0][tid];
#pragma unroll
            for (int u = 1; u < STREAMS; ++u) merge_stats(mm, zz, sm[half][u][tid], sz[half][u][tid]);
            float *o = part + (((long)h * nchunks + chunk0 + at) * R_total + row_base + tid) * 2;
            o[0] = mm;
            o[1] = zz;
        }
    };
    int at = 0, tiles_in = 0;   // chunk being summed, tiles of it that are in
    auto before_tile = [&] {    // the chunk that ended with the tile before this one
        if (MANY && at > 0 && tiles_in == 0) store(at - 1, (at - 1) & 1);
    };
    auto after_tile = [&] {
        if (MANY && ++tiles_in == chunk_keys / TK) {
            park(at & 1);
#pragma unroll
            for (int b = 0; b < NBW; ++b) { m[b] = -INFINITY; z[b] = 0.f; }
            ++at;
            tiles_in = 0;
        }
    };

    // Two accumulator sets: the products of tile t are issued between the softmax instructions of
    // tile t - 1, so that the matrix core works while the vector unit does the exponentials.
    f32x16 acc[2][NBW];
    // the kSteps * NBW matrix instructions of one tile; between(j) is placed after the j-th
    auto multiply = [&](const bf16x8 (&kc)[kSteps], int set, auto &&between) {
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int b = 0; b < NBW; ++b) {   // rows = keys, columns = queries
                acc[set][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kc[s], q[b][s], s == 0 ? zero : acc[set][b], 0, 0, 0);
                between(s * NBW + b);
            }
    };
    // running (max, sum) of the lane's queries updated with tile t, whose products are in `set`
    auto finish = [&](int t, int set) {
        const int kb = k0 + TK * t + kBlk * stream;
        if (kb + kBlk <= P) {   // every key of the block is a prefix key: visible to all rows
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                float tm = acc[set][b][0];
#pragma unroll
                for (int i = 1; i < 16; ++i) tm = fmaxf(tm, acc[set][b][i]);
                const float mn = fmaxf(m[b], tm * c);
                float zz = z[b] * fast_exp2(m[b] - mn);
#pragma unroll
                for (int i = 0; i < 16; ++i) zz += fast_exp2(fmaf(acc[set][b][i], c, -mn));
                m[b] = mn;
                z[b] = zz;
            }
        } else {                // the block touches the window (or the end of the head): mask
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                float tm = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (kb + acc_row(i, hh) <= last_vis[b]) tm = fmaxf(tm, acc[set][b][i]);
                const float mn = fmaxf(m[b], tm * c);
                if (mn != -INFINITY) {
                    float zz = z[b] * fast_exp2(m[b] - mn);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (kb + acc_row(i, hh) <= last_vis[b]) zz += fast_exp2(fmaf(acc[set][b][i], c, -mn));
                    m[b] = mn;
                    z[b] = zz;
                }
            }
        }
    };
    auto head = [&](const unsigned char *buf) {
        bf16x8 kc[kSteps];
        tile_read(buf, stream, l32, hh, kc);
        multiply(kc, 0, [](int) {});
    };
    auto body = [&](const unsigned char *buf, int t, int set) {
        before_tile();
        bf16x8 kc[kSteps];
        tile_read(buf, stream, l32, hh, kc);
        const int kb = k0 + TK * (t - 1) + kBlk * stream;   // the block finished here
        if (kb + kBlk <= P) {
            // the same arithmetic as finish(), in the same order, cut into slices: the row maxima
            // while the LDS reads are on their way, then two exponentials after every matrix
            // instruction (the scheduling barriers keep the compiler from regrouping them)
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                float tm = acc[set ^ 1][b][0];
#pragma unroll
                for (int i = 1; i < 16; ++i) tm = fmaxf(tm, acc[set ^ 1][b][i]);
                const float mn = fmaxf(m[b], tm * c);
                z[b] = z[b] * fast_exp2(m[b] - mn);
                m[b] = mn;
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(kc, set, [&](int j) {
                constexpr int per = 16 / kSteps;   // NBW * 16 values over NBW * kSteps instructions
#pragma unroll
                for (int e = per * j; e < per * j + per; ++e)
                    z[e / 16] += fast_exp2(fmaf(acc[set ^ 1][e / 16][e % 16], c, -m[e / 16]));
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            multiply(kc, set, [](int) {});
            finish(t - 1, set ^ 1);
        }
        after_tile();
    };
    if constexpr (NBW <= 2) {
        GKV_TILE_PIPELINE_OVERLAPPED(TK, NT, ONCE, Kh, k0, k1 - 1, 1, ntile, queries(), head, body, finish);
    } else {   // three row blocks per wave: a second accumulator set does not fit the registers
        auto one_tile = [&](const unsigned char *buf, int t) {
            before_tile();
            bf16x8 kc[kSteps];
            tile_read(buf, stream, l32, hh, kc);
            multiply(kc, 0, [](int) {});
            finish(t, 0);
            if (t + 1 < ntile) after_tile();
        };
        GKV_TILE_PIPELINE_TK(TK, NT, ONCE, Kh, k0, k1 - 1, 1, ntile, queries(), one_tile);
    }

    park(at & 1);
    __syncthreads();
    before_tile();   // (a chunk that ended with the last tile but one)
    store(at, at & 1);
}

// ---------------------------------------------------------------- pass B ---
// votes: PERQ = false: [Hkv * vote_rows, P], row h*vote_rows + vote_row_base + g holds
// the sum over the query rows of row group g; PERQ = true: [Hkv * G, P], one row per
// query head (needs every query head's rows inside one row group).
//
// Heads with more than 128 stacked query rows are handled in parts of at most 128
// rows (row_base .. row_base + R of R_total), one launch per part: the keys are then
// streamed once per part.
//
// pool_half >= 0 (all rows of a head in one workgroup): the votes never leave the workgroup.  Each row
// group (max pooling: each query head) keeps the votes of the workgroup's keys in LDS, the workgroup also multiplies the
// pool_half keys on either side of its chunk, and at the end it writes the pooled, grouped
// scores of its chunk itself: votes[] is then the score array [Hkv, P].  The sums are
// formed in the order of the separate pooling kernel, so the bits are the same.
template <int NB, int SPLIT, bool PERQ, int STREAMS, bool ONCE>
__global__ __launch_bounds__(64 * STREAMS * SPLIT) void score_votes_kernel(
    const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ Qw, int N, int P, int w, int G,
    int chunk_keys, float c, const float *__restrict__ part, int part_chunks,
    float *__restrict__ votes, int R_total, int R_real, int row_base, int vote_rows, int vote_row_base,
    int pool_half)
{
    constexpr int R = NB * kBlk, NBW = NB / SPLIT, NT = 64 * STREAMS * SPLIT, TK = kBlk * STREAMS;
    extern __shared__ __align__(16) unsigned char kt[];   // two key tiles
    __shared__ float bias_s[R];
    const int h = blockIdx.y, chunk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
    const int stream = wv % STREAMS, grp = wv / STREAMS, row0 = grp * NBW * kBlk;

    const int k0 = chunk * chunk_keys, k1 = min(P, k0 + chunk_keys);
    if (k0 >= P) return;
    const bool fused = pool_half >= 0;
    const int first = fused ? max(0, k0 - pool_half) : k0;      // keys this workgroup multiplies
    const int kend = fused ? min(P, k1 + pool_half) : k1;
    const int span = chunk_keys + 2 * pool_half;
    // [row groups, or query heads][span], slot 0 = key k0 - pool_half
    float *vs = reinterpret_cast<float *>(kt + 2 * TK * kPitch);
    if (fused)   // outside the row: zeros (average), nothing (max)
        for (int u = tid; u < (PERQ ? G : SPLIT) * span; u += NT) vs[u] = PERQ ? -INFINITY : 0.f;

    bf16x8 q[NBW][kSteps];
    const uint16_t *Qh = Qw + (long)h * R_real * kD;
    float bias[NBW][16];
    auto statistics = [&] {
        {   // Row statistics of the whole head: merge the chunks of pass A, PARTS threads per row, each a run
            // of chunks whose loads leave eight at a time.  (One thread per row and one load after the
            // other was the longest part of the kernel's start with few heads: 25.4 us with 32 chunks, 21 us now.)
            constexpr int PARTS = NT / R;
            __shared__ float2 stat_s[PARTS][R];
            const int row = tid % R, pt = tid / R, per = (part_chunks + PARTS - 1) / PARTS;
            const int cb = min(pt * per, part_chunks), ce = min(cb + per, part_chunks);
            float mm = -INFINITY, zz = 0.f;
            if (pt < PARTS) {
                for (int c0 = cb; c0 < ce; c0 += 8) {
                    float2 o[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        o[u] = *reinterpret_cast<const float2 *>(
                            part + (((long)h * part_chunks + min(c0 + u, ce - 1)) * R_total + row_base + row) * 2);
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (c0 + u < ce) merge_stats(mm, zz, o[u].x, o[u].y);
                }
                stat_s[pt][row] = make_float2(mm, zz);
            }
            __syncthreads();
            if (tid < R) {
                mm = stat_s[0][tid].x;
                zz = stat_s[0][tid].y;
#pragma unroll
                for (int u = 1; u < PARTS; ++u) merge_stats(mm, zz, stat_s[u][tid].x, stat_s[u][tid].y);
                // zz >= 1: the row maximum itself contributes exp2(0); rows that only fill a block vote zero
                bias_s[tid] = row_base + tid < R_real ? mm + __log2f(zz) : INFINITY;
            }
        }
    };
    auto queries = [&] {   // (its barriers make bias_s known to all)
        spread_rows<NT, R, 2 * TK>(kt, tid, row0, [&](int x) { return Qh + (long)min(row_base + x, R_real - 1) * kD; }, q,
                                   statistics);
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) bias[b][i] = bias_s[row0 + kBlk * b + acc_row(i, hh)];
    };

    const uint16_t *Kh = Kc + (long)h * N * kD;
    const int ntile = (kend - first + TK - 1) / TK;
    const int bpq = PERQ ? w / kBlk : 1;   // MFMA row blocks per query head

    auto multiply_tile = [&](const unsigned char *buf, int t) {
        bf16x8 kc[kSteps];
        tile_read(buf, stream, l32, hh, kc);

        f32x16 acc[NBW];
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int b = 0; b < NBW; ++b)   // rows = queries, columns = keys
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[b][s], kc[s], acc[b], 0, 0, 0);

        float pb[NBW];
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) s += fast_exp2(fmaf(acc[b][i], c, -bias[b][i]));
            pb[b] = s;
        }
        const int key = first + TK * t + kBlk * stream + l32;
        if constexpr (!PERQ) {
            float p = pb[0];
#pragma unroll
            for (int b = 1; b < NBW; ++b) p += pb[b];
            p = add_other_half(p);
            if (hh == 0 && key < kend) {
                if (fused) vs[grp * span + key - (k0 - pool_half)] = p;
                else votes[((long)h * vote_rows + vote_row_base + grp) * P + key] = p;
            }
        } else {
            const int g0 = (row_base / kBlk + grp * NBW) / bpq;   // first query head of this row group
#pragma unroll
            for (int g = 0; g < NBW; ++g) {
                float p = 0.f;
#pragma unroll
                for (int b = 0; b < NBW; ++b) p += (b / bpq == g) ? pb[b] : 0.f;
                p = add_other_half(p);
                if (g0 + g < G && g * bpq < NBW && hh == 0 && key < kend) {
                    if (fused) vs[(g0 + g) * span + key - (k0 - pool_half)] = p;
                    else votes[((long)h * G + g0 + g) * P + key] = p;
                }
            }
        }
    };
    GKV_TILE_PIPELINE_TK(TK, NT, ONCE, Kh, first, kend - 1, 1, ntile, queries(), multiply_tile);
    if (fused) {
        __syncthreads();
        if constexpr (PERQ) {   // max pooling: per query head, then the sum over the heads
            for (int o = tid; o < k1 - k0; o += NT) {
                float total = 0.f;
                for (int g = 0; g < G; ++g) {
                    float best = -INFINITY;
                    for (int t = 0; t <= 2 * pool_half; ++t) best = fmaxf(best, vs[g * span + o + t]);
                    total += best;
                }
                votes[(long)h * P + k0 + o] = total / (float)G;
            }
            return;
        }
        // votes of a key summed over the row groups (in group order, into group 0's array), then the
        // taps of every output in key order: the additions of the separate pooling kernel
        if (SPLIT > 1) {
            for (int u = tid; u < span; u += NT) {
                float v = 0.f;
#pragma unroll
                for (int g = 0; g < SPLIT; ++g) v += vs[g * span + u];
                vs[u] = v;
            }
            __syncthreads();
        }
        const float taps = (float)(2 * pool_half + 1), div = (float)G;
        for (int o = tid; o < k1 - k0; o += NT) {
            float acc = 0.f;
            if (pool_half == 3) {
#pragma unroll
                for (int t = 0; t < 7; ++t) acc += vs[o + t];
            } else {
                for (int t = 0; t <= 2 * pool_half; ++t) acc += vs[o + t];
            }
            votes[(long)h * P + k0 + o] = acc / taps / div;
        }
    }
}

// Keys per workgroup of the votes pass.  A compute unit runs one of these workgroups at a time (208
// registers a lane, eight waves), and every workgroup pays for its queries, its first tiles and the merge
// of the statistics -- about as long as 256 keys take.  So the cut with the fewest keys per compute unit
// wins, counting whole rounds of 256 workgroups: for few heads as many chunks as one round takes, for
// many as few as keep the rounds full.  At most `most` keys: the votes of a chunk sit in LDS beside the
// key tiles, one row per row group (two, or four at 256 query rows) or query head; at least two tiles, as the
// pooling window's halo is read twice.  (1024 workgroups of at least 1024 keys before, chunks of 6144 with 256 query rows; us, before /
// now: 8 heads of 4096 keys 18.0 / 13.6, of 16384 21.0 / 16.3, of 65536 51 / 31; 128 heads of 8192 76 / 51;
// 8 heads of 32768 keys with 256 query rows 103 / 28.)
constexpr int kComputeUnits = 256;
int votes_chunk_keys(int Hkv, int N, int rows, int lds_rows)
{
    const int least = 256, most = rows == 256 ? 6144 : (lds_rows <= 2 ? 8192 : 16384 / lds_rows / 128 * 128);
    const int cmin = (N + most - 1) / most, cmax = (N + least - 1) / least > cmin ? (N + least - 1) / least : cmin;
    long best = -1;
    int keys = 0;
    auto consider = [&](long chunks) {
        const long c = chunks < cmin ? cmin : (chunks > cmax ? cmax : chunks);
        const long ck = ((N + c - 1) / c + 127) / 128 * 128;
        const long rounds = ((long)Hkv * ((N + ck - 1) / ck) + kComputeUnits - 1) / kComputeUnits;
        const long cost = rounds * (ck + 256);
        if (best < 0 || cost < best) { best = cost; keys = (int)ck; }
    };
    consider(cmin);
    const long r0 = ((long)Hkv * cmin + kComputeUnits - 1) / kComputeUnits;
    for (long r = r0; r < r0 + 4; ++r) consider(r * kComputeUnits / Hkv);
    return keys;
}

// Keys per workgroup of the statistics pass: 512 workgroups of at least 1024 keys (twice as long as the votes
// pass's: they hold no votes in LDS, and every workgroup pays for its queries and its first tiles), or one round of
// at least one tile each while 1024 keys would leave compute units idle (8 heads of 4096 keys 16.9 -> 10.2 us,
// of 16384 17.5 -> 13.8).  Larger launches keep 512 workgroups: one round of twice as many keys is up to
// a fifth faster for mid sizes, but a lane's sum of exponentials then runs over twice as many terms in 32
// bits (error of the scores against 64 bits at 256 heads of 32768 keys 1.5e-6 -> 2.4e-6).
int stats_keys(int Hkv, int N)
{
    const long total = (long)Hkv * N;
    long ck = (total + 511) / 512, least = (total + kComputeUnits - 1) / kComputeUnits;
    least = least < 128 ? 128 : (least > 1024 ? 1024 : least);
    if (ck < least) ck = least;
    return (int)((ck + 127) / 128 * 128);                     // 4 waves x 32 keys
}

}  // namespace

// Query rows of a head as the kernels take them: whole blocks of 32, and 256 rather than two parts when
// there are more than 128 and the votes may mix query heads (one pass over the keys at 256 rows costs less
// than two at 128 and the rest: 32 layers of 4 heads x 224 rows x 16384 keys, the whole pass 752 -> 549 us).
int mfma_score_rows(int G, int w, int per_qhead_votes)
{
    const int R = (G * w + kBlk - 1) / kBlk * kBlk;
    return R > 128 && !per_qhead_votes ? 256 : R;
}

// A sum of exponentials depends in its last bits on where the keys are cut.  A batch cuts them as one of its
// layers alone would, a workgroup taking several chunks, so that both give the same scores -- but for launches of
// more than 2^19 keys (heads x tokens) with whole 32-row blocks, which are cut by all their heads: a workgroup
// then has one chunk and the votes pass two to merge (32 layers of 8 heads x 32768 keys).  Parking a chunk
// and the votes pass's longer merge cost 1 to 4 % of a small batch (whole pass, us, cut by all heads / by a
// layer's: 8 layers of 8 heads x 4096 keys 86.2 / 89.5, 4 x 8 x 8192 86.3 / 88.8, 32 x 4 x 16384 of 112 rows 385 / 391).
constexpr long kLayerCutKeys = 1L << 19;

MfmaScorePlan mfma_score_plan(int Hkv, int layer_heads, int G, int w, int N, int per_qhead_votes)
{
    MfmaScorePlan pl;
    const bool as_layer = (long)Hkv * N <= kLayerCutKeys || G * w % kBlk != 0;
    pl.chunk_keys = stats_keys(as_layer ? layer_heads : Hkv, N);
    pl.chunks = (N + pl.chunk_keys - 1) / pl.chunk_keys;
    // as many workgroups a head as the heads of the launch ask for, evenly filled
    const int all = stats_keys(Hkv, N), wgs = (N + all - 1) / all;
    pl.per_wg = pl.chunks > wgs ? (pl.chunks + wgs - 1) / wgs : 1;
    pl.part_bytes = (size_t)Hkv * pl.chunks * mfma_score_rows(G, w, per_qhead_votes) * 2 * sizeof(float);
    return pl;
}

namespace {

// The stacked query rows of a head are cut into parts of at most 128 rows; a part of
// nb 32-row blocks runs with 2 row groups per key stream when nb is even (and, for
// per-query-head votes, every query head stays inside one group), else with 1.
int part_rows(int R_total, int part) { return R_total - 128 * part < 128 ? R_total - 128 * part : 128; }
int part_split(int rows, int w, int per_qhead_votes)
{
    const int nb = rows / 32;
    if (nb % 2) return 1;
    if (per_qhead_votes && (w / 32) > nb / 2) return 1;
    return 2;
}

}  // namespace

// Rows of the votes array per KV head.
int mfma_score_vote_rows(int G, int w, int per_qhead_votes)
{
    if (per_qhead_votes) return G;
    const int R = mfma_score_rows(G, w, per_qhead_votes);
    int rows = 0;
    for (int part = 0; 128 * part < R; ++part) rows += part_split(part_rows(R, part), w, 0);
    return rows;
}

template <int NB, int SPLIT, int STREAMS>
static hipError_t launch_stats_nb(const uint16_t *K, const uint16_t *Q, int Hkv, int N, int P, int w,
                                  const MfmaScorePlan &plan, float c, float *part, int R_total, int R_real, int row_base,
                                  hipStream_t st)
{
    const dim3 grid((plan.chunks + plan.per_wg - 1) / plan.per_wg, Hkv), block(64 * STREAMS * SPLIT);
    const size_t lds = 2 * (kBlk * STREAMS) * kPitch;
    const bool once = reads_past_caches((size_t)Hkv * N * kD * 2);
    auto *kernel = plan.per_wg > 1 ? (once ? score_stats_kernel<NB, SPLIT, STREAMS, true, true> : score_stats_kernel<NB, SPLIT, STREAMS, true, false>)
                                   : (once ? score_stats_kernel<NB, SPLIT, STREAMS, false, true> : score_stats_kernel<NB, SPLIT, STREAMS, false, false>);
    if (!allow_big_lds((const void *)kernel)) return hipGetLastError();
    hipLaunchKernelGGL(kernel, grid, block, lds, st, K, Q, N, P, w, plan.chunk_keys, plan.chunks, plan.per_wg, c, part,
                       R_total, R_real, row_base);
    return hipGetLastError();
}

hipError_t launch_mfma_score_stats(const void *Kc, const void *Qw, int Hkv, int layer_heads, int Hq, int N, int w,
                                  float scale, int per_qhead_votes, float *part, hipStream_t st)
{
    const int G = Hq / Hkv, R_real = G * w, R = mfma_score_rows(G, w, per_qhead_votes), P = N - w;
    const MfmaScorePlan plan = mfma_score_plan(Hkv, layer_heads, G, w, N, per_qhead_votes);
    const float c = scale * 1.4426950408889634f;
    const uint16_t *K = (const uint16_t *)Kc, *Q = (const uint16_t *)Qw;
    if (R == 256)   // one workgroup takes all 256 rows: 2 key streams x 4 row groups, tiles of 64 keys
        return launch_stats_nb<8, 4, 2>(K, Q, Hkv, N, P, w, plan, c, part, R, R_real, 0, st);
    // other row counts beyond 128: parts of at most 128 rows, one launch per part
    for (int pt = 0; 128 * pt < R; ++pt) {
        hipError_t err = hipErrorInvalidValue;
        switch (part_rows(R, pt) / 32) {
            case 1: err = launch_stats_nb<1, 1, 4>(K, Q, Hkv, N, P, w, plan, c, part, R, R_real, 128 * pt, st); break;
            case 2: err = launch_stats_nb<2, 2, 4>(K, Q, Hkv, N, P, w, plan, c, part, R, R_real, 128 * pt, st); break;
            case 3: err = launch_stats_nb<3, 1, 4>(K, Q, Hkv, N, P, w, plan, c, part, R, R_real, 128 * pt, st); break;
            case 4: err = launch_stats_nb<4, 2, 4>(K, Q, Hkv, N, P, w, plan, c, part, R, R_real, 128 * pt, st); break;
        }
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

template <int NB, int SPLIT, int STREAMS = 4>
static void launch_votes_nb(dim3 grid, const uint16_t *K, const uint16_t *Q, int N, int P, int w, int G,
                            int ck, float c, const float *part, int chunks, int per_q, float *votes,
                            int R_total, int R_real, int row_base, int vote_rows, int vote_row_base, int pool_half,
                            hipStream_t st)
{
    const size_t lds = 2 * (kBlk * STREAMS) * kPitch + (pool_half >= 0 ? (size_t)(per_q ? G : SPLIT) * (ck + 2 * pool_half) * 4 : 0);
    const bool once = reads_past_caches((size_t)grid.y * N * kD * 2);
    auto *kernel = per_q ? (once ? score_votes_kernel<NB, SPLIT, true, STREAMS, true> : score_votes_kernel<NB, SPLIT, true, STREAMS, false>)
                         : (once ? score_votes_kernel<NB, SPLIT, false, STREAMS, true> : score_votes_kernel<NB, SPLIT, false, STREAMS, false>);
    if (!allow_big_lds((const void *)kernel)) return;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * STREAMS * SPLIT), lds, st, K, Q, N, P, w, G, ck, c, part, chunks, votes, R_total,
                       R_real, row_base, vote_rows, vote_row_base, pool_half);
}

// Widest pooling window of the votes pass: its halo is multiplied twice and sits in LDS beside the chunk.
constexpr int kFusedPool = 129;

bool mfma_score_fuses_pool(int G, int w, int per_qhead_votes, int pool_kernel)
{
    const int R = mfma_score_rows(G, w, per_qhead_votes);
    return (R <= 128 || (R == 256 && !per_qhead_votes)) && pool_kernel <= kFusedPool;
}

hipError_t launch_mfma_score_votes(const void *Kc, const void *Qw, int Hkv, int layer_heads, int Hq, int N, int w,
                                  float scale, int per_qhead_votes, int fused_pool_kernel,
                                  const float *part, float *votes, hipStream_t st)
{
    const int G = Hq / Hkv, R_real = G * w, R = mfma_score_rows(G, w, per_qhead_votes), P = N - w;
    const MfmaScorePlan plan = mfma_score_plan(Hkv, layer_heads, G, w, N, per_qhead_votes);
    // fused pooling: a workgroup also multiplies pool_half keys on either side of its chunk; the
    // P prefix keys are spread evenly over the chunks
    const int pool_half = fused_pool_kernel > 0 ? (fused_pool_kernel - 1) / 2 : -1;
    const int vck = votes_chunk_keys(Hkv, N, R, pool_half >= 0 && per_qhead_votes ? G : 2), vchunks = (N + vck - 1) / vck;
    const int ck = pool_half >= 0 ? (P + vchunks - 1) / vchunks : vck;
    const float c = scale * 1.4426950408889634f;
    const uint16_t *K = (const uint16_t *)Kc, *Q = (const uint16_t *)Qw;
    const dim3 grid(vchunks, Hkv);
    const int vote_rows = mfma_score_vote_rows(G, w, per_qhead_votes);
    int vote_row_base = 0;
    if (R == 256 && !per_qhead_votes) {   // all rows in one workgroup (see the statistics pass): four row groups
        launch_votes_nb<8, 4, 2>(grid, K, Q, N, P, w, G, ck, c, part, plan.chunks, 0, votes, R, R_real, 0, vote_rows, 0,
                                 pool_half, st);
        return hipGetLastError();
    }
#define GKV_VOTES(NB, SP)                                                                             \
    launch_votes_nb<NB, SP>(grid, K, Q, N, P, w, G, ck, c, part, plan.chunks, per_qhead_votes, votes, R, \
                            R_real, row_base, vote_rows, vote_row_base, pool_half, st)
    for (int pt = 0; 128 * pt < R; ++pt) {
        const int row_base = 128 * pt, rows = part_rows(R, pt);
        const int split = part_split(rows, w, per_qhead_votes);
        switch (rows / 32) {
            case 1: GKV_VOTES(1, 1); break;
            case 2: if (split == 2) GKV_VOTES(2, 2); else GKV_VOTES(2, 1); break;
            case 3: GKV_VOTES(3, 1); break;
            case 4: if (split == 2) GKV_VOTES(4, 2); else GKV_VOTES(4, 1); break;
            default: return hipErrorInvalidValue;
        }
        vote_row_base += split;
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
#undef GKV_VOTES
    return hipGetLastError();
}

}  // namespace gkv
