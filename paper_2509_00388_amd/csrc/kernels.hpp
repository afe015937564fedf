// Host-side launchers of the GraphKV kernels.  Every launcher only enqueues
// work on `st` and returns hipGetLastError() of its launches.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace gkv {

// Kernels that use more than 64 KiB of dynamic LDS need a one-time opt-in per kernel and
// device.  Which (device, kernel) pairs have it is the library's only state besides the
// measurement aid; it is process-wide and guarded by a mutex, so first calls may come from
// several host threads at once.  Returns false if the opt-in failed.
bool allow_big_lds(const void *kernel, int bytes = 160 * 1024 - 8192);

// Whether a call's keys are too many for a pass over them to leave behind what the next pass could find in the 256 MiB
// of the memory-side cache: then they are loaded (and large outputs stored) without a claim to a place in the caches,
// which leaves the L2 to lists that are written a few bytes at a time.  (Whole pass, us, with a claim / without: heads
// of 32K keys, 8 of them (64 MiB) 144 / 150, 24 260 / 274, 32 278 / 279, 48 417 / 398, 64 468 / 431, 128 840 / 755; key
// norms of 8000 keys, 64 heads (125 MiB) 121 / 125, 128 193 / 190, 256 372 / 325; one score call of 128 MiB 103 / 117, of
// 256 MiB 103 / 117, of 384 MiB 177 / 179.)
inline bool reads_past_caches(size_t key_bytes) { return key_bytes > (size_t)256 << 20; }

// ---- selection (select.hip) -------------------------------------------------
// For each of `rows` rows of x (row r starts at x + r*ld, n entries): the k entries that come first
// by (value descending, index ascending), written in ascending index order to idx_out + r*idx_ld
// (and their values to val_out + r*val_ld when val_out != nullptr).
hipError_t launch_topk_rows(const float *x, long ld, int n, int rows, int k, int32_t *idx_out, long idx_ld,
                            float *val_out, long val_ld, hipStream_t st);

// Source nodes (Eq. 2) plus the X nodes ranked right behind them: src [rows, S] gets the S
// best entries of each row (ascending index), ext [rows, S + X] the same S followed by the next
// X (ascending index), by (value descending, index ascending).  S + X <= n, S + X <= kMaxExtSources.
hipError_t launch_pick_sources(const float *x, long ld, int n, int rows, int S, int X, int32_t *src,
                               int32_t *ext, hipStream_t st);

// Neighbourhoods of the heads whose overflow flag is set (filter route, bf16, d = 128): a fixed
// number of workgroups walk the (head, source) rows of those heads, each computing one row of
// edges into its own scratch row (rows: redo_rows_scratch_bytes()) and taking the exact top-m.
size_t redo_rows_scratch_bytes(int heads, int S, int P);
hipError_t launch_redo_rows(const void *Ac, const void *Kc, int heads, int N, int P, int S, int m, const int32_t *src,
                            const int32_t *overflow, float *rows, int32_t *nbr, float *nbr_e, hipStream_t st);

// ---- scalar kernels for any dtype / shape (generic.hip) ----------------------
// logits [Hq*w, N] (fp32, scaled), then per-row max and sum of exp.
hipError_t launch_generic_logits(const void *Kc, const void *Qw, int dtype, int Hkv, int Hq, int d,
                                 int N, int w, float scale, float *logits, float *row_max,
                                 float *row_sum, hipStream_t st);
// votes [Hq, P]: softmax weights summed over the window rows; rows of `pitch` logits, row statistics `step` apart.
hipError_t launch_generic_votes(const float *logits, int pitch, const float *row_max, const float *row_sum, int step,
                                int Hq, int P, int w, float *votes, hipStream_t st);
// E [Hkv, S, P] cosine of row src[h,a] of Ac against every prefix row of Kc; self = -inf.
// (Eq. 1: Ac = Kc = keys; other pairings of tensors give the Discussion's other edges.)
hipError_t launch_generic_cosine(const void *Ac, const void *Kc, int dtype, int Hkv, int d, int N, int P, int S,
                                 const int32_t *src, float *E, hipStream_t st);
// scores[h,j] = -||k_j||
hipError_t launch_knorm(const void *Kc, int dtype, int Hkv, int d, int N, int P, float *scores,
                        hipStream_t st);

// ---- the same contractions on the matrix cores, any dtype / shape (gemm.hip) ----------
struct GemmScorePlan {
    int chunk_keys, chunks;   // keys per chunk, chunks per head of the row statistics
    int per_wg;               // chunks a workgroup takes
    int pitch;                // logits kept per row
    size_t part_bytes;        // bytes of per-chunk row statistics, 0 for a single chunk
};
// Hkv: heads of the launch; layer_heads: KV heads of one of its layers.
GemmScorePlan gemm_score_plan(int Hkv, int layer_heads, int G, int w, int N, bool trim);
// logits [Hq*w, pitch] (fp32, scaled) and part [Hkv, chunks, G*w] (max, sum of exp) over visible keys.
hipError_t launch_gemm_logits(const void *Kc, const void *Qw, int dtype, int Hkv, int Hq, int d, int N, int w,
                              float scale, const GemmScorePlan &pl, float *logits, float *part, hipStream_t st);
// scores [Hkv, P] from logits and the row statistics of `chunks` chunks, votes, pooling and the mean over
// the group included (gemm_votes_pools(pool_kernel)).  launch_gemm_merge makes one chunk of many, stat
// [Hq*w] (max, sum): in front of it where there are many (gemm_merges_first), and in front of
// launch_generic_votes and launch_pool_group, which wider pooling windows take.
bool gemm_votes_pools(int pool_kernel);
bool gemm_merges_first(const GemmScorePlan &pl, int rows);   // rows: stacked query rows per KV head
hipError_t launch_gemm_merge(const float *part, const GemmScorePlan &pl, int Hkv, int Hq, int w, float *stat,
                             hipStream_t st);
hipError_t launch_gemm_votes(const float *logits, const GemmScorePlan &pl, const float *part, int chunks, int Hkv,
                             int layer_heads, int Hq, int N, int w, int pool_kernel, int pool_mode, float *scores,
                             hipStream_t st);
// Same contract as launch_generic_cosine.
hipError_t launch_gemm_cosine(const void *Ac, const void *Kc, int dtype, int Hkv, int d, int N, int P, int S,
                              const int32_t *src, float *E, hipStream_t st);

// ---- pooling, signal propagation, gather (stages.hip) -----------------------
// votes [Hkv*Gv, P] -> scores [Hkv, P]: pool each of the Gv rows of a head, sum, divide by div.
hipError_t launch_pool_group(const float *votes, int Hkv, int Gv, int P, int pool_kernel,
                             int pool_mode, float div, float *scores, hipStream_t st);
// Eq. 5 for one round: scores[h, nbr] *= prod (1 -/+ alpha e), ascending source order.
hipError_t launch_decay(float *scores, int Hkv, int P, int S, int m, const int32_t *nbr,
                        const float *nbr_e, float alpha, int signal, hipStream_t st);
// An update that the next kernel with a workgroup per head does first (decay.hpp): items = triples per
// thread as decay_rides_along() says, 0: none.
struct DecayArgs {
    const int32_t *nbr;
    const float *nbr_e;
    int items, count;
    float alpha;
    int signal;
};
int decay_rides_along(int P, int S, int m);
// Kout[q,t,:] = Kc[q, idx[q,t], :] for the heads q of a batch, same for V; packed
// outputs, per-layer budgets from the plan; row_bytes multiple of 16.
hipError_t launch_gather(const void *Kc, const void *Vc, const int32_t *idx, int heads, int N,
                         const LayerPlan &plan, int max_budget, int row_bytes, void *Kout, void *Vout,
                         hipStream_t st);
// Final selection of a batch: row q keeps budget[l] - w entries and writes them,
// followed by the window tokens P .. P + w - 1, to its packed idx row.
// (An update that rides along changes the scores first.)  scratch: topk_final_scratch_bytes() bytes, with which
// few long rows are shared out to many workgroups (0: none is used), or nullptr.
// gather: Kout null, or the retained rows are copied too (topk_final_gathers()).
struct GatherArgs {
    const void *Kc, *Vc;
    void *Kout, *Vout;
    int N, row_bytes;
};
bool topk_final_gathers(int P, int max_budget, int row_bytes);
size_t topk_final_scratch_bytes(int rows, int P);
hipError_t launch_topk_final(float *scores, int P, int rows, const LayerPlan &plan, int w, int32_t *idx,
                             const DecayArgs &update, const GatherArgs &gather, void *scratch, hipStream_t st);
hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, long n, hipStream_t st);
hipError_t launch_copy_f32(const float *src, float *dst, long n, hipStream_t st);

// ---- bf16 MFMA kernels, d = 128 (mfma_score.hip, mfma_cosine.hip) ----------
struct MfmaScorePlan {
    int chunk_keys, chunks;   // keys per chunk, chunks per head of the row statistics
    int per_wg;               // chunks a workgroup of the statistics pass takes
    size_t part_bytes;        // bytes of per-chunk row statistics
};
int mfma_score_rows(int G, int w, int per_qhead_votes);   // stacked query rows, filled up to what the kernels take
// Hkv: heads of the launch; layer_heads: KV heads of one of its layers.
MfmaScorePlan mfma_score_plan(int Hkv, int layer_heads, int G, int w, int N, int per_qhead_votes);
// Pass A: per (head, chunk, row) partial max and sum of exp2 over the chunk's visible keys.
// Pass B: votes [Hkv * rows, P] with rows = mfma_score_vote_rows(): partial sums over
// groups of query rows (to be added up), or one row per query head.
int mfma_score_vote_rows(int G, int w, int per_qhead_votes);
hipError_t launch_mfma_score_stats(const void *Kc, const void *Qw, int Hkv, int layer_heads, int Hq, int N, int w,
                                  float scale, int per_qhead_votes, float *part, hipStream_t st);
// fused_pool_kernel > 0 (only if mfma_score_fuses_pool()): pooling with that kernel size and the
// mean over the query heads are done in the same kernel; `votes` is then the
// score array [Hkv, P] and no pooling kernel follows.
bool mfma_score_fuses_pool(int G, int w, int per_qhead_votes, int pool_kernel);
hipError_t launch_mfma_score_votes(const void *Kc, const void *Qw, int Hkv, int layer_heads, int Hq, int N, int w,
                                  float scale, int per_qhead_votes, int fused_pool_kernel,
                                  const float *part, float *votes, hipStream_t st);
// E [Hkv, S, P] from bf16 keys (same contract as launch_generic_cosine).
hipError_t launch_mfma_cosine(const void *Ac, const void *Kc, int Hkv, int N, int P, int S, const int32_t *src,
                              float *E, hipStream_t st);
// Neighbourhoods without the dense block (see mfma_cosine.hip):
bool mfma_filter_applies(int P, int m, long rows);   // rows: heads x sources of the launch
int mfma_sample_cols(int P);          // keys in the strided sample
int mfma_bound_rank(int m, int stride);   // rank in the sample at which a row's bound is taken (<= m)
int mfma_cand_cap(int P, int m);      // candidates per source the exact select can take
bool source_reuse_applies(int S);     // lists can be kept from round to round
constexpr int kSpecRows = 32;         // speculative rows per head: one or two MFMA row blocks of 32
constexpr int kMaxExtSources = 256;   // largest S + kSpecRows the source selection splits
// Geometry of the filter route for one call.  The per-row buffers (tau [Hkv, pitch], cand
// [Hkv, pitch, row_slots] x 8 bytes, cand_cnt [Hkv, pitch, chunk_slots]) hold, per head,
// the S sources of the first round, then X speculative rows (the nodes ranked right behind the
// sources: the likeliest new sources of later rounds, whose candidate lists the first round's
// pass builds on the side).  New sources of later rounds that have no kept list reuse rows 0 .. S - 1.
struct MfmaFilterPlan {
    int S, X;
    int sb;           // 32-row groups per workgroup in the passes over the full source list
    int pitch;        // S + X
    int chunk_cols;   // keys per workgroup of the filter pass
    int chunks;       // workgroups (= candidate slices) per head and source group
    int slice_cap;    // entries per (row, chunk) slice
    int late_cols, late_chunks, late_slice_cap;   // the same for the passes over new sources of later rounds
    int chunk_slots;  // slice sizes a row has room for (cand_cnt)
    long row_slots;   // entries a row has room for (cand), at least chunks * slice_cap
    int cand_cap;     // entries the exact select can take per row
};
// short_slices: no more memory for candidates than keys in no particular order need.
MfmaFilterPlan mfma_filter_plan(int Hkv, int P, int S, int m, bool keep_lists, bool speculate, bool short_slices);
size_t mfma_bound_scratch_bytes(int Hkv, int P, const MfmaFilterPlan &g);   // what chunks of the sample leave (0 if one chunk)
// Whether the first round's filter pass takes the bounds itself: the bound pass is then left out.
bool mfma_filter_takes_bounds(int P, int m, const MfmaFilterPlan &g);
// Bound pass: tau = a value that at least m of the row's edges reach (but for about one row in
// 10^7, which the select notices), from the edges to every (P / sample_cols)-th key; clears
// overflow [Hkv].  first_round: src is the extended list
// [Hkv, S + X] (all rows in use, rows 0 .. of the buffers); otherwise src is the list of new
// sources [Hkv, S], n_src [Hkv] of them in use, rows 0 .. of the buffers.
hipError_t launch_mfma_cosine_bound(const void *Ac, const void *Kc, int Hkv, int N, int P, int m,
                                    const MfmaFilterPlan &g, bool first_round, const int32_t *src,
                                    const int32_t *n_src, void *hist_part, float *tau, int32_t *overflow,
                                    hipStream_t st);
// Filter pass: streams all keys; edges that reach a row's tau go to its slices, their number
// per slice to cand_cnt.  Same source lists, rows and hist_part (first round) as the bound pass.
hipError_t launch_mfma_cosine_filter(const void *Ac, const void *Kc, int Hkv, int N, int P, int m,
                                     const MfmaFilterPlan &g, bool first_round, const int32_t *src,
                                     const int32_t *n_src, const void *hist_part, const float *tau, void *cand,
                                     int32_t *cand_cnt, int32_t *overflow, hipStream_t st);
// From the second round on (match.hpp): which sources keep their list from the round before (copied
// from prev_nbr / prev_e to nbr / nbr_e), which are speculative rows of the first round (the last X
// entries of ext [Hkv, S + X]; not used for heads that overflowed then: spec_bad [Hkv], set by the first
// match of a call from the first round's overflow flags), and which need another bound and filter pass
// (new_src [Hkv, S], n_new [Hkv]).  sel_row / sel_pos [Hkv, S], n_sel [Hkv]: the selections to
// run as (candidate row, source slot).
struct MatchArgs {
    int S, X, m, first;
    const int32_t *prev_src, *prev_nbr;
    const float *prev_e;
    int32_t *nbr;
    float *nbr_e;
    const int32_t *ext;
    int32_t *overflow;   // [Hkv] flags of the round before, cleared for this one by launch_pick_match()
    int32_t *spec_bad, *new_src, *n_new, *sel_row, *sel_pos, *n_sel;
};
// Source nodes (Eq. 2) of a later round and their match, one launch for S <= 256 (pick_match_applies).
bool pick_match_applies(int S);
hipError_t launch_pick_match(float *x, int n, int rows, const MatchArgs &a, int32_t *src, const DecayArgs &update,
                             hipStream_t st);
hipError_t launch_match_sources(const MatchArgs &a, const int32_t *cur, int Hkv, hipStream_t st);
// Exact top-m over candidate rows -> nbr / nbr_e [Hkv, S, m]; skips heads with overflow[h], and
// raises overflow[h] itself if a row has more candidates than it can take.  rows == nullptr:
// candidate row x -> source slot x for all S sources of src [Hkv, S]; otherwise the listed ones.
struct SelectRows {
    const int32_t *n_rows;   // [Hkv] selections per head
    const int32_t *row;      // [Hkv, S] candidate row of the x-th selection
    const int32_t *pos;      // [Hkv, S] its source slot in this round's list
};
hipError_t launch_nbr_select(const void *cand, const int32_t *cand_cnt, int32_t *overflow, const int32_t *src,
                             int Hkv, int m, const MfmaFilterPlan &g, const SelectRows *rows, int32_t *nbr,
                             float *nbr_e, hipStream_t st);
// A later round's bound and filter passes in one launch, for few heads (overflow is not cleared).
bool late_filter_applies(int Hkv, const MfmaFilterPlan &g);
hipError_t launch_late_filter(const void *Ac, const void *Kc, int Hkv, int N, int P, int m, const MfmaFilterPlan &g,
                              const int32_t *new_src, const int32_t *n_new, void *cand, int32_t *cand_cnt,
                              int32_t *overflow, hipStream_t st);

}  // namespace gkv
