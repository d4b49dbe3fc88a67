// Host-side plan and the launchers each kernel file exports to the API file.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/vatt.h"
#include "../../include/vatt_testing.h"
#include "vatt_dev.h"

namespace vatt {

constexpr int kSubTile = 8;            // keys per sub-tile maximum
constexpr int kHeadThreads = 512;      // workgroup size of the per-head kernel
constexpr int kHeadThreadsLong = 1024; // ... for rows whose 8-key maxima do not fit the registers of 512 threads
constexpr int kGatherThreads = 256;
// Targets N and SDPA: the doubles that the budget kernel leaves of a head for the merge, D_f and then N_f.  They take the place of the
// flags of the head's own draws made ahead, which the kernel has read by then.
constexpr int kFixedStride = kHeadThreads * sizeof(uint32_t) / sizeof(double);
static_assert(1 + 128 <= kFixedStride, "a column each");
// Launch orders of the score pass (see the score kernel); the values of VATT_OPT_SCORE_ORDER.
constexpr int kScoreOrderTile = 0, kScoreOrderKvHead = 1, kScoreOrderBlocks = 2;
constexpr int kDenseThreads = 256;
constexpr int kCapacityMax = 170752;   // tokens per sequence: what the selection kernel's LDS bitmaps are sized for
constexpr int kCacheSlotsMax = 8192;   // slots of the random cache of base-sample rows, per (sequence, KV head)

// What the per-head kernel leaves for the gather kernel.
struct HeadRec {
  float m;        // max score of the head
  float scale;    // n_s / b (0 when b == 0)
  int32_t n, n_sink, n_win, k, b, n_s;
  int32_t b_keep;  // leading entries of the final sample that repeat the base sample (nested samples), else 0
  int32_t base_cached;  // the base sample's entries are slots of the random cache (their rows are read from it)
  int32_t tail_by_token;  // the gather reads the sampled tokens' scores from the score row by token (else, like
                          // those of sink, window and top-k, from where the selection kernel left them: at the
                          // list places)
};

// Workgroups of a head that take part, of the `splits` the grid has for it: no more than its list fills with steps.
// A workgroup costs a chain of about four memory round trips however few rows it has, and the lengths of the lists are
// only known here: with all 16 of them 8 sequences of 0.5K - 7K tokens (497 rows a head) took 16.7 us, with as many as there
// are steps of 128 rows 9.4 us, with two for each step 11; long lists are as fast as before (16 x 32K tokens, 1867 rows: 40 us,
// 6.1 TB/s of V rows).  One that takes part alone writes the result itself.
__device__ __forceinline__ int used_splits(int splits, int total, int step_rows) {
  return min(splits, (total + step_rows - 1) / step_rows);
}

// Whether the rows of a list are read with ordinary loads instead of non-temporal ones: `vectors` query vectors share a KV head
// and run on one XCD (all of a group in the order of head_of_block, else one per query token), and where their lists, each
// about as long as this one, together are as long as half the sequence, a row that one has fetched is found in the L2 by others.
// Measured (gather kernel, us, non-temporal -> ordinary, and the listed rows of all vectors over the length): 1 x 32K tokens with
// 16 query tokens 41.5 -> 31.2 (3.6), 8 22.3 -> 20.0 (1.8), 4 13.4 -> 11.6 (0.9); 1 x 128K with 4 37.1 -> 36.1 (0.9), 8 x 32K with
// lists of 0.2 of it 78.4 -> 75.7 (0.8); but 8 x 32K with lists of 0.06 to 0.12 31.8 -> 32.7 (0.25 - 0.5), 16 x 32K 41.0 -> 44.7
// (0.2), 4 x 128K 29.4 -> 32.8 (0.2), and 1 x 91K with 4 KV heads, their 8 vectors on as many XCDs, and 3 query tokens 44.8 -> 48.0
// (0.3 on each).
// The line is `quarters` / 4.  The gather of the caller-supplied path, which reads K and V rows of the drawn tokens, none of which the
// vectors share, takes 3 where they are whole groups of several heads: at 2 several sizes were slower than without ordinary loads (whole
// step, us, without / at 2 / at 3: 16 x 16K at epsilon 0.02 112.3 / 113.4 / 111.5, with the random cache 108.6 / 112.2 / 107.5, 32 x 3K
// 79.0 / 79.9 / 75.5, 2 x 32K with 3 query tokens 60.4 / 61.6 / 56.6, 8 x 16K with 2 82.4 / 86.5 / 83.2; though 16 x 4K 48.2 / 44.8 / 45.9,
// 24 x 4K 61.7 / 57.6 / 59.7).  Where they are the query tokens of one head it stays at 2 (1 x 59K with 6 119.4 / 108.0 / 114; 17 x 0.3K -
// 5K with 2, 16 KV heads of 64 columns, at 2 50.8, at 3 51.8).
__device__ __forceinline__ bool rows_are_shared(int total, int vectors, int n, int quarters = 2) {
  return 4ll * total * vectors > (long long)quarters * n;
}

constexpr int kDenseKeys = 32;  // keys a wave of the matrix-core dense kernel takes at a time
// Waves of a dense matrix-core workgroup that take different query vectors (32 each) of the same keys, and the keys of its
// waves together, the unit in which keys are dealt out to workgroups.
inline int dense_vector_waves(int vectors) { return vectors <= 32 ? 1 : vectors <= 64 ? 2 : 4; }
inline int dense_unit(int vectors) { return kDenseKeys * (kDenseThreads / 64) / dense_vector_waves(vectors); }
inline int dense_rounds(int vectors) { return (vectors + 127) / 128; }  // workgroups for all vectors of a KV head
inline bool dense_dots(int q_len, int group) { return q_len == 1 && group <= 2; }  // too few vectors for the matrix cores
constexpr int kDenseSplitsMax = 128;

struct Plan {
  vatt_params p;
  int device;         // -1: geometry only
  int num_cus;
  int group;          // Hq / Hkv
  int q_len;          // query tokens per sequence and call (1: single-token decoding)
  int vbatch;         // batch * q_len: every (sequence, query token) pair is handled like a sequence of its own
  float sm_scale;
  double z_half;      // Phi^{-1}(1 - delta/2)
  double range_factor;  // > 0: the range-based Hoeffding budget, ln(2 / delta) / 2 (denominator target)
  double z_quarter;   // Phi^{-1}(1 - delta/4)
  double eps, cap_frac;
  SelectParams sel;
  // sizes
  int n_pad;          // score row stride (floats)
  int n_sub;          // sub-tiles of kSubTile keys per row (the score kernel leaves each one's largest score)
  int k_max, b0_max, b_max;
  int head_threads;   // workgroup size of the per-head kernel
  int split_cap;  // upper bound of the four split counts below that share the partial-sum regions
  int gather_splits, dense_splits, vstat_splits, given_splits;
  int dense_share;  // dense kernel: workgroups per KV head that the keys of the batch are dealt out to (0: equal splits)
  int given_fuse_splits;  // caller-supplied top-k: > 0, the second selection phase also gathers, with this many workgroups per head
  int sparse_splits;  // workgroups per head of the score kernel of the listed tokens when it only writes scores
  size_t idx_cap;
  int64_t seg_off[5];
  size_t head_lds_bytes;
  int topk_general_path;          // test hook: the top-k selection always takes its general path
  int sampler_small_batches;      // test hook: the sampler works in batches of 256 draws only
  uint32_t sampler_draw_cap;      // draws after which a sample is completed in index order (0: 64 L + 4096)
  int group_major;                // the later kernels launch the query heads of a KV head on one XCD (head_of_block)
  int score_order;                // launch order of the score pass (kScoreOrder*)
  int nested_samples;             // the final sample keeps the base sample and extends it (not the paper's fresh draw)
  int ascending_samples;          // the samples' index lists are written in ascending token order
  int budget_multiple;            // the budget is rounded up to a multiple of this (1: the paper's rule)
  int prework;                    // the sampler streams' first batches are made by workgroups of the score launch
  int fuse_splits;                // > 0: the selection kernel also gathers, with this many workgroups per head
  int cache_slots;                // slots per (sequence, KV head) of the random cache of base-sample rows
  // workspace offsets (bytes)
  size_t off_scores, off_sub_max, off_sparse, off_head_rec, off_gather_part,
      off_debug, off_vstat_part, off_dense_part, off_pre_tok, off_pre_flags, off_base_slot, ws_bytes;
  KVLayout kv_k, kv_v;  // templates; base pointers are passed per call
};

// Caller-supplied top-k, gather apart: workgroups per head that gather I_f beside the second selection phase, in its launch (0: the
// gather behind it takes the whole list).  The host knows the plan's capacity, not the lengths: the lines lie where they do for sequences
// of about that length.  Whole step, us, behind -> beside:
// Heads: where every head's phase has a compute unit to itself, 128 heads of 128K tokens 101.3 -> 94.9, 192 of 12K 34.5 -> 33.0; with more
// of them the rows wait for slots and the launch takes as long as the two one after the other, 512 heads of 32K 111.0 -> 113.2, 1024 of
// 0.3K - 1.5K paged 61.3 -> 65.4.  Where query tokens share the rows two phases on a unit still gain on longer rows: 512 heads of 9K (16
// query tokens) 58.9 -> 54.7, 32K with lists of 0.2 of it 219 -> 195; but of 1.5K with such lists 38.8 -> 40.5, 960 of 3K 84.9 -> 86.2.
// Rows: below some 400 the two launches are as long as they were, 192 heads of 1.5K (293 rows) 26.2 -> 26.6, of 6K (406) 31.4 -> 30.9; with
// few heads, whose phases are shorter, 32 of 4K (356) 24.4 -> 24.9, of 0.9K (526) 22.8 -> 23.5, of 16K (656) 22.9 -> 22.8.
// Budgets: where (z / epsilon)^2 is large beside the length the sample is most of the residual, the phase takes long and the rows saved are
// few: 192 heads of 9K at epsilon 0.005 78.2 -> 81.9, 512 at 0.01 135.3 -> 137.5, but 192 of 30K at 0.01 129.7 -> 124.4.  So it
// is with the targets N and SDPA, by the values: 128 heads of 9K 91.7 -> 94.0, of 32K at epsilon 0.2 71.7 -> 67.9.
// Workgroups: up to 6 per head and some two per unit in all, with 4 steps each at most; more of them slow the phases beside them (256
// heads of 30K with 2 / 4 58.6 / 61.3, 192 of 24K with 2 / 4 44.7 / 45.4, 32 of 100K with 6 / 11 39.2 / 41.2), and fewer steps than
// a list has are idle launches.
// Sequences far shorter than a long capacity lose up to 2 %, longer ones gain: 512 heads (16 query tokens), capacity 32K, of 1K 48.3 -> 49.2,
// 2K 59.6 -> 60.5, 3K 68.1 -> 68.3, 4K 75.4 -> 74.4, 6K 84.7 -> 82.9, 24K 179.7 -> 171.0.
constexpr int kFixedLeast = 400, kFixedLeastFew = 640, kFixedWorkgroups = 576, kFixedMost = 6;
__host__ __device__ constexpr int fixed_step_rows(int head_dim) { return kHeadThreads / (head_dim / 8) * 8; }  // rows of one of them per step
constexpr int given_part_slots(const Plan& pl) { return pl.split_cap > 16 ? pl.split_cap : 16; }  // partial sums of a head in all
constexpr int given_fixed_splits(const Plan& pl) {
  const int heads = pl.vbatch * pl.p.n_q_heads, step = fixed_step_rows(pl.p.head_dim);
  const int rows = pl.p.sink + pl.p.window + pl.k_max;
  if (heads > pl.num_cus && (pl.q_len == 1 || heads > 2 * pl.num_cus || pl.p.n_max < 4096)) return 0;
  if (pl.p.target != VATT_TARGET_D || rows < (2 * heads > pl.num_cus ? kFixedLeast : kFixedLeastFew)) return 0;
  if ((pl.z_half / pl.eps) * (pl.z_half / pl.eps) > 4.0 * pl.p.n_max) return 0;
  const int steps = (rows + step - 1) / step;
  int splits = kFixedWorkgroups / heads;
  splits = splits > kFixedMost ? kFixedMost : splits < 2 ? 2 : splits;
  splits = splits < (steps + 3) / 4 ? (steps + 3) / 4 : splits > steps ? steps : splits;
  const int left = given_part_slots(pl) - (pl.given_splits < given_part_slots(pl) ? pl.given_splits : given_part_slots(pl) - 1);
  return splits < left ? splits : left;
}
// Workgroups per head of the gather behind it.
constexpr int given_tail_splits(const Plan& pl) {
  return given_fixed_splits(pl) > 0 && pl.given_splits >= given_part_slots(pl) ? given_part_slots(pl) - 1 : pl.given_splits;
}

inline double* fixed_sums_of(const Plan& pl, void* ws) { return reinterpret_cast<double*>(static_cast<char*>(ws) + pl.off_pre_flags); }

// Bytes of score rows a call writes, and the size from which on they are taken to outgrow the last-level cache beside
// what else passes through it.
inline size_t score_bytes(const Plan& pl) { return (size_t)pl.vbatch * pl.p.n_q_heads * pl.p.n_max * sizeof(float); }
constexpr size_t kScoreBytesLarge = 32000000;

// Every launcher returns a hipError_t from hipGetLastError() after the launch.
// seq_seeds: needed (may be nullptr otherwise) when score_prework(pl)
hipError_t launch_score(const Plan& pl, const void* q, const void* k, const int32_t* block_table,
                        const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws, hipStream_t st);
// The score pass of a multi-query step (q_len > 1): all query tokens and group heads share one read of K.
hipError_t launch_score_chunk(const Plan& pl, const void* q, const void* k, const int32_t* block_table,
                              const int32_t* seq_lens, void* ws, hipStream_t st);
// phase 0: everything (target D); phase 1: through the base sample.
hipError_t launch_head(const Plan& pl, int phase, const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws,
                       int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                       hipStream_t st);
// The path with a caller-supplied top-k set: selection phase 0 (sets, base sample) and 1 (budget, final sample),
// scores of the listed tokens, gather with the final sample's scores computed on the way.
// Selection and gather in one kernel for small batches (denominator target, fresh final sample), then the merge
// of the per-workgroup partial sums.
hipError_t launch_head_fused(const Plan& pl, const void* v, const int32_t* block_table, const int32_t* seq_lens,
                             const uint64_t* seq_seeds, void* ws, int32_t* out_idx, int32_t* out_counts,
                             double* out_budget_raw, float* out_stats, float* out_o, float* out_lse, bool pre_made,
                             hipStream_t st);
// Whether workgroups of the score launch make the sampler streams' first batches for the fused selection kernel
// (single-token steps only).
inline bool score_prework(const Plan& pl) {
  return pl.prework && pl.fuse_splits > 0 && !pl.nested_samples && !pl.ascending_samples && pl.q_len == 1 &&
         pl.p.target == VATT_TARGET_D;
}
hipError_t launch_gather_merge(const Plan& pl, void* ws, int splits, float* out_o, float* out_lse, hipStream_t st);
int fused_splits_for(const Plan& pl);           // the plan's own choice (0: separate kernels)
bool fused_splits_fit(const Plan& pl, int splits);  // whether the fused kernel can run with that many
// rcache (may be nullptr): random cache the base sample is taken from when it holds enough residual tokens;
// the score kernel of the listed tokens then reads those tokens' rows from the cache.
hipError_t launch_given_select(const Plan& pl, const int32_t* seq_lens, const uint64_t* seq_seeds,
                               const int32_t* given_idx, const int32_t* given_cnt, const void* rcache, void* ws,
                               int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                               hipStream_t st);
// The second selection phase with the gather fused in (small batches, denominator target, fresh final sample),
// followed by the merge of the per-workgroup partials.
// (phase 0: first selection phase plus the scores of I_f and I_bs; phase 1: second phase plus the gather)
hipError_t launch_given_fused(const Plan& pl, int phase, const void* q, const void* k, const void* v,
                              const int32_t* block_table, const int32_t* seq_lens, const uint64_t* seq_seeds,
                              const int32_t* given_idx, const int32_t* given_cnt, const void* rcache, void* ws,
                              int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                              hipStream_t st);
// The second selection phase, with the gather of I_f beside it in the same launch where given_fixed_splits says so.
hipError_t launch_given_budget(const Plan& pl, const void* v, const int32_t* block_table, const int32_t* seq_lens,
                               const uint64_t* seq_seeds, void* ws, int32_t* out_idx, int32_t* out_counts, double* out_budget_raw,
                               float* out_stats, hipStream_t st);
hipError_t launch_given_merge(const Plan& pl, void* ws, int splits, float* out_o, float* out_lse, hipStream_t st);
int given_fused_splits_for(const Plan& pl);
bool given_fused_fits(const Plan& pl, int splits);
// (with targets N and SDPA it also reads the V rows of the listed tokens and leaves the numerator statistics)
hipError_t launch_sparse_score(const Plan& pl, const void* q, const void* k, const void* v,
                               const int32_t* block_table, const void* rcache, void* ws, const int32_t* out_idx,
                               hipStream_t st);
// Random cache of base-sample rows: layout for a plan, state after the tokens of existing sequences have
// arrived one by one, append of one token per sequence with its arrival in the cache, token lists for tests.
CacheLayout cache_layout(const Plan& pl);
hipError_t launch_cache_fill(const Plan& pl, const void* k, const void* v, const int32_t* block_table,
                             const int32_t* seq_lens, const uint64_t* cache_seeds, void* rcache, hipStream_t st);
hipError_t launch_append_cached(const Plan& pl, const void* k_new, const void* v_new, void* k, void* v,
                                const int32_t* block_table, int32_t* seq_lens, const uint64_t* cache_seeds,
                                void* rcache, hipStream_t st);
hipError_t launch_cache_read(const Plan& pl, const void* rcache, int32_t* out_tok, int32_t* out_count,
                             hipStream_t st);
hipError_t launch_given_gather(const Plan& pl, const void* q, const void* k, const void* v,
                               const int32_t* block_table, void* ws, const int32_t* out_idx, float* out_o,
                               float* out_lse, hipStream_t st);
hipError_t launch_vstats(const Plan& pl, const void* v, const int32_t* block_table, void* ws,
                         const int32_t* out_idx, hipStream_t st);
// Targets N and SDPA: budget and final sample, behind phase 1 and the V-side statistics.
hipError_t launch_budget(const Plan& pl, const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws, int32_t* out_idx,
                         int32_t* out_counts, double* out_budget_raw, float* out_stats, hipStream_t st);
hipError_t launch_gather(const Plan& pl, const void* v, const int32_t* block_table, void* ws,
                         const int32_t* out_idx, float* out_o, float* out_lse, hipStream_t st);
hipError_t launch_dense(const Plan& pl, const void* q, const void* k, const void* v, const int32_t* block_table,
                        const int32_t* seq_lens, void* ws, float* out_o, float* out_lse, hipStream_t st);
hipError_t launch_append(const Plan& pl, const void* k_new, const void* v_new, void* k, void* v,
                         const int32_t* block_table, int32_t* seq_lens, hipStream_t st);
hipError_t set_kernel_attributes(const Plan& pl);        // every selection kernel: dynamic LDS limit
hipError_t set_budget_kernel_attributes();
hipError_t set_given_kernel_attributes(const Plan& pl);  // (its part for the caller-supplied-top-k kernels)
// Dynamic and static LDS of the selection kernels, and the LDS list entries of the fused gathers.
size_t head_kernel_lds_bytes(int n_max, int head_threads);
size_t head_kernel_static_lds_bytes();
int fused_dlist_cap(const Plan& pl, int splits);
// Reads `bytes` (a multiple of 16) from src and discards them; sink is 4 KiB of device memory.
hipError_t launch_stream_read(const void* src, size_t bytes, void* sink, hipStream_t st);
// Reads the 256-byte rows rows[0 .. count) (row numbers, clamped into [0, rows_total)) of src and discards them.
hipError_t launch_row_read(const void* src, size_t rows_total, const int32_t* rows, size_t count, void* sink,
                           hipStream_t st);

}  // namespace vatt

struct vatt_plan {
  vatt::Plan pl;
};
