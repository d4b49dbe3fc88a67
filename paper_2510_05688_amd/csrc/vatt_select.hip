// Index selection and budget: Algorithm 1 up to the final sample and all of Algorithm 2, per (sequence, query head),
// in one kernel with one workgroup per head.
//
// Top-k: the k largest scores of the middle region, ties to the lower token, i.e. the k smallest composites
// (~order_key(score), token).  Usual path: the score kernel leaves the largest score of every 8 keys; the k-th
// largest of those maxima is a lower bound of the k-th largest score (located to one bin of a 2048-bin LDS
// histogram), the 8-key sub-tiles that reach it are listed, their scores loaded, and the scores at or above the
// bound are the candidates, a few more than k.  The members among them: histogram over 2048 equal-width score
// bins, the bin that holds rank k located by a workgroup scan, the bins before it taken whole and its few scores
// ranked as composites.  General path (short rows, very large k, long runs of equal scores): the same histogram selection
// streamed over the whole row, refined by further histograms over the integer keys when a bin holds many
// scores, and by token order inside a run of equal scores, so the result is exact for any data.
//
// Samples: sequential uniform draws from the middle region (Philox4x32-10 words, unbiased multiply-and-reject
// mapping), skipping top-k members and tokens drawn before; the first c accepted tokens are the sample (for
// c > n_s / 2 they are the tokens left out).  The kernel processes the draw sequence in batches: all draws of
// a batch are generated at once, repeated tokens are resolved to their earliest draw, and a prefix count in
// draw order finds where the sample is complete; the result equals the sequential procedure bit for bit.
//
// What bounds it: a workgroup is one dependency chain of barriers and trips to global memory, and with few heads the chain is the time:
// with the gather fused in, one head of 1K tokens 12.6 us, 32 heads of 32K 19.5, 256 heads of 0.5K - 7K 20.5 (rows of 32K have more
// maxima and candidates to pass through the same steps).  Where workgroups fill the chip they also wait for their scattered reads (scores
// of the proposals, sub-tiles of the candidates): 512 heads of 32K tokens 29 - 34 us, 1024 heads of 1K - 32K 54.
//
// Floating-point sums are taken in a fixed order, or as fixed-point integers where the order depends on
// scheduling, so the statistics and the budget are reproducible too.
#include "vatt_select.h"

namespace vatt {
namespace {

// NT = workgroup size.  FD = 0: selection only (the gather is a kernel of its own).  FD = head dimension: fused
// gather for small batches, where one workgroup per head would leave most of the chip idle and every kernel
// boundary is a visible part of the step: every head gets A.splits workgroups (blockIdx.z), each of which runs
// the whole selection (identical results in all of them: nothing is exchanged), keeps every A.splits-th token
// of the head's list in LDS, gathers those V rows and leaves a partial (sum w V, sum w) for the merge kernel.
// Only workgroup 0 of a head writes the index lists, counts, statistics and budget.  The rows of I_f are
// requested as soon as the top-k set is known and are added after the samplers have run.
// ALONE: one workgroup per head, which writes the head's result itself (a branch on A.splits at the end cost the others
// 0.4 us, and the split arithmetic these 1.4 us).
// PHASE: 0 everything (denominator target), 1 through the base sample (targets N and SDPA; budget_kernel has the rest).
// OPTIONS: a plan with an option set that the usual call does without (head_options) has a kernel of its own; without them the
// selection-only kernel, which is at its register limit, takes 33.6 instead of 36.5 us for 16 x 32K tokens, the fused one 20.0 instead
// of 20.4 for 1 x 32K and 12.7 instead of 13.4 for one head of 1K.
// PAIR: two workgroups per head (head_pair).  A form of its own, too: as a run-time branch it made the forms with one workgroup per head
// spill, which then took (whole call, us, branch -> form of its own) 263.0 -> 262.4 for 8 x 64K tokens, 145.2 -> 143.6 for 6 x 40K at
// epsilon 0.02, 89.1 -> 88.1 for 1 x 32K with 16 query tokens; and with two workgroups 4 x 128K 250.3 -> 249.3, 1 x 60K 57.5 -> 56.8.
template <int NT, int FD, bool PAGED, bool ALONE, int PHASE, bool OPTIONS, bool PAIR>
__global__ __launch_bounds__(NT, FD > 0 ? 1 : 4) void head_kernel(HeadArgs A) {
  touch_args<HeadArgs>();
  if constexpr (FD > 0 || !OPTIONS) A.nested = A.ascending = 0;  // (in the fused kernel too: what it does not serve has no code there, 0.3 us)
  if constexpr (!OPTIONS) {
    A.topk_general = A.small_batches = 0;
    A.range_factor = 0.0;
    A.b_multiple = 1;
  }
  if constexpr (PHASE == 0) A.target = VATT_TARGET_D;
  constexpr bool kFused = FD > 0;
  using O = HeadOps<NT>;
  using TKR = TopkOps<NT, RowView<NT>>;
  using TKC = TopkOps<NT, CandView<NT>>;
  using HeadSmem = typename O::HeadSmem;
  using Sampler = typename O::Sampler;
  constexpr int SW = NT / kWave;
  extern __shared__ __align__(16) unsigned char dyn_smem[];
  __shared__ TopkSmem ts;
  const int h = head_of_block((int)blockIdx.x, A.Hq, A.Hkv, A.group_major), b = blockIdx.y;
  const int bh = b * A.Hq + h;
  const int tid = threadIdx.x;
  constexpr bool kSplit = kFused && !ALONE;
  const uint32_t split = kSplit ? blockIdx.z : 0u, shift = kSplit ? (uint32_t)A.split_shift : 0u;
  const uint32_t smask = (1u << shift) - 1u;
  // PAIR: the second workgroup of a head repeats the top-k step and writes what the first would make the base sample wait for, the
  // lists of I_f, and what it would make the budget wait for: the scores of the final sample's proposals at the list places (long rows)
  // or the budget kernel's first batch of draws.  Nothing is exchanged: it writes the scores of all accepted draws of the
  // first batch, and the first workgroup says in the record whether the sample is the beginning of them.  A compute unit takes
  // four to five clocks per scattered 4-byte read, and with one workgroup per head half of the units pulled all of them.
  // Whole call, us, one -> two: 4 x 128K tokens 250.4 -> 244.1, 1 x 128K 112.1 -> 102.3, 2 of 9K - 100K paged 108.5 -> 99.1, 4 x 50K with
  // k and b0 of 5 % 152.0 -> 145.8, 1 x 60K at epsilon 0.02 59.2 -> 56.4, 1 x 91K with 3 query tokens 108.9 -> 98.4.
  // Targets N and SDPA: 4 x 16K 82.5 -> 80.5, 1 x 32K 86.8 -> 84.4, 2 x 9K of 16 heads 50.7 -> 47.8, 4 x 128K 333 -> 327, 1 x 100K 155 -> 152.7.
  static_assert(!PAIR || (!kFused && !OPTIONS && (NT >= 1024 || PHASE == 1)), "what head_pair asks for");
  const bool second = PAIR && blockIdx.z == 1u;
  const bool lister = !PAIR || second;              // this workgroup writes the lists of I_f
  const bool writer = split == 0u && !second;       // this workgroup writes the head's other outputs
  // The sub-tile maxima the score kernel left are requested first of all, before even the sequence length is
  // known (what lies beyond the row's own sub-tiles is masked once it is): the kernel starts with a chain of
  // dependent loads, and this takes one link out of it.  Rows of up to 8 * NT sub-tiles keep the maxima in
  // registers for the three passes below, longer rows stream them in every pass.
  constexpr int SU = NT >= 1024 ? 16 : 8;  // sub-tile maxima a thread has in flight (rows up to 131072 / 32768 tokens)
  const float* sub_max = A.sub_max + (int64_t)bh * A.n_sub;
  float sub_reg[SU];
#pragma unroll
  for (int u = 0; u < SU; ++u) {
    const int t = u * NT + tid;
    sub_reg[u] = t < A.n_sub ? sub_max[t] : -INFINITY;
  }
  uint4 pre_t = make_uint4(0u, 0u, 0u, 0u);
  uint32_t pre_f = 0u;
  bool pre_made = false;
  if (NT == kHeadThreads && PHASE == 0 && A.pre_tok) {
    pre_t = A.pre_tok[(int64_t)bh * NT + tid];
    pre_f = A.pre_flags[(int64_t)bh * NT + tid];
    pre_made = pre_made_of(A.pre_flags[(int64_t)bh * NT]);  // one word for the whole workgroup: uniform
  }
  // In a multi-query step b stands for (sequence, query token); query token t of q_len sees the sequence up to
  // and including itself, which leaves out the q_len - 1 - t newer tokens.
  const int seq = seq_of_pair(b, A.q_len), qtok = b - seq * A.q_len;
  const int n = max(min(max(A.seq_lens[seq], 1), A.n_max) - (A.q_len - 1 - qtok), 1);  // clamp, then the causal cut
  const HeadSizes hs = head_sizes(n, A.sp);
  const int words_max = bitmap_words(A.n_max);
  const int words = (n + 31) >> 5;

  HeadSmem& sm = *reinterpret_cast<HeadSmem*>(dyn_smem);
  // (the 512-thread kernel can generate the first batches of both streams at once: the final sample's stream
  // then needs a scratch bitmap and mail slots of its own)
  constexpr bool kTwoStreams = NT == kHeadThreads;
  const HeadLds at = head_lds<NT, kTwoStreams>(A.n_max);
  uint32_t* lds = reinterpret_cast<uint32_t*>(dyn_smem);
  uint64_t* cand = reinterpret_cast<uint64_t*>(lds + at.cand);
  uint32_t *qual = lds + at.qual, *bm_f = lds + at.bm_f, *taken0 = lds + at.taken0, *taken1 = lds + at.taken1;
  uint32_t *scratch = lds + at.scratch0, *scratch1 = lds + at.scratch1, *wpre = lds + at.wpre, *mail = lds + at.mail0, *mail1 = lds + at.mail1;
  // Histogram of the candidates' scores: in the mail slots of the final sample's stream, once its first batch is made.
  static_assert(kMailSlots == kBins, "the histogram takes the place of the mail slots");
  uint32_t* cand_hist = mail1;
  // fused gather: this workgroup's share of I_f and of the final sample, and the cross-wave sums
  uint32_t* glist = lds + at.lists;
  uint32_t* dlist = glist + (kFused ? A.glist_cap : 0);
  // (the scores of the listed tokens, so that the gather requests V rows only)
  float* glist_sc = reinterpret_cast<float*>(dlist + (kFused ? A.dlist_cap : 0));
  float* dlist_sc = glist_sc + (kFused ? A.glist_cap : 0);
  float* g_red = dlist_sc + (kFused ? A.dlist_cap : 0);
  // (I_f is dealt out in runs of consecutive list places: its top-k part is in ascending token order, so a
  // workgroup's rows then lie close together in the cache)
  uint32_t g_lo = 0, g_hi = 0;
  if (kFused) {
    const uint32_t n_f = (uint32_t)(hs.n_sink + hs.n_win + hs.k);
    const uint32_t run = min((n_f + smask) >> shift, (uint32_t)A.glist_cap);  // ceil(n_f / splits)
    g_lo = min(split * run, n_f);
    g_hi = min(g_lo + run, n_f);
  }
  // What the lists in LDS know a row by: its token, or on a paged cache its place in the pool (pages in front of its own times
  // the page, plus the place in it; a pool that fits the memory has fewer than 2^32).  The block-table entries are asked for
  // where the tokens become known, long before the lists are written, so that the rows do not wait for them: 8 x 0.5K - 7K
  // tokens 36.8 -> 35.1 us per call.
  constexpr bool kCode = kFused && PAGED;
  auto code_of = [&](uint32_t tok, int blk) {
    if constexpr (!kCode) return tok;
    else return ((uint32_t)min(max(blk, 0), A.L.num_blocks - 1) << A.L.page_shift) + (tok & ((1u << A.L.page_shift) - 1u));
  };
  auto row_code = [&](uint32_t tok) { return code_of(tok, kv_block<kCode>(A.L, seq, (int)tok)); };
  auto to_glist = [&](uint32_t p, uint32_t code, float sc) {
    if (kFused && p >= g_lo && p < g_hi) {
      glist[p - g_lo] = code;
      glist_sc[p - g_lo] = sc;
    }
  };

  const float* row = A.scores + (int64_t)bh * A.n_pad;
  int32_t* idx = A.out_idx + (int64_t)bh * A.idx_cap;
  // Selection-only kernel: where a list is written with the scores at hand (sink, window, top-k, and a final
  // sample that the first batch of draws holds) they are left at the list places, so that the gather kernel reads
  // them next to the list entries instead of from the score row by token.  A sample made another way is read by
  // token (HeadRec.tail_by_token).
  float* place_sc = A.place_sc + (int64_t)bh * A.idx_cap;
  const uint64_t seed = A.seq_seeds[seq];

  VATT_STAMP(A.dbg, 0);
  // The score row is requested first (when it is kept in registers), so that its latency overlaps the
  // sampler work below.
  RowView<NT> rv;
  rv.row = row;
  rv.n = n;
  const float edge0 = tid < hs.n_sink ? row[tid] : -INFINITY;
  const float edge1 = tid < hs.n_win ? row[hs.mid_hi + tid] : -INFINITY;
  const int edge0_blk = kv_block<kCode>(A.L, seq, min(tid, n - 1));
  const int edge1_blk = kv_block<kCode>(A.L, seq, min(hs.mid_hi + tid, n - 1));
  const uint32_t row0_code = row_code(0u);
  // cleared: the bitmaps bm_f .. scratch1, which follow each other, and the first histogram
  for (int w = tid; w < (kTwoStreams ? 5 : 4) * (words_max / 4); w += NT)
    reinterpret_cast<uint4*>(bm_f)[w] = make_uint4(0u, 0u, 0u, 0u);
  for (int w = tid; w < kBins / 4; w += NT) reinterpret_cast<uint4*>(ts.hist)[w] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) {
    ts.cand_n = 0;
    ts.qual_n = 0;
    ts.slist_n = 0;
  }
  __syncthreads();

  // The draw sequences do not depend on the scores: the first batch of each stream is generated, and the
  // scores of the base-sample proposals are requested, before the top-k set is known.
  const uint32_t L = (uint32_t)max(hs.mid_hi - hs.mid_lo, 1);
  Sampler S0, S1;
  S0.taken = taken0;
  S0.scratch = scratch;
  S0.mail = mail;
  S0.bm_f = bm_f;
  S0.wpre = wpre;
  S0.row = row;
  S0.seed = seed;
  S0.stream = 0u;
  S0.head = (uint32_t)h;
  S0.query = (uint32_t)qtok;
  S0.L = L;
  S0.thr = (uint32_t)((0x100000000ull - (uint64_t)L) % (uint64_t)L);
  {
    const uint64_t dflt = 64ull * (uint64_t)L + 4096ull;
    S0.cap = (uint32_t)min(A.draw_cap ? (uint64_t)A.draw_cap : dflt, 0x80000000ull);
  }
  S0.m = 0.f;
  S0.dbg = A.dbg ? A.dbg + 200 : nullptr;
  S1 = S0;
  S1.taken = taken1;
  S1.scratch = scratch1;
  S1.mail = mail1;
  S1.stream = 1u;
  S1.dbg = A.dbg ? A.dbg + 300 : nullptr;
  DrawBatch spec0 = {}, spec1 = {};
  const bool want0 = hs.n_s > 0 && hs.b0 < hs.n_s && !second;
  const bool want1 = hs.n_s > 0 && (PHASE != 1 || (NT >= 1024 && second)) && !A.nested;  // (a nested final sample rarely draws at all)
  const int n_sub = (n + kSubTile - 1) / kSubTile;
  const int sub_lo = (hs.mid_lo + kSubTile - 1) / kSubTile, sub_hi = hs.mid_hi / kSubTile;  // whole middle sub-tiles
  const bool sub_resident = n_sub <= SU * NT;
#pragma unroll
  for (int u = 0; u < SU; ++u) {
    const int t = u * NT + tid;
    sub_reg[u] = (sub_resident && t < n_sub) ? sub_reg[u] : -INFINITY;
  }
  // g(maxima[SU], first sub-tile of the batch): slot u is sub-tile first + u * NT + tid, -inf beyond the row
  auto each_sub_batch = [&](auto&& g) {
    if (sub_resident) {
      g(sub_reg, 0);
    } else {
      for (int base = 0; base < n_sub; base += NT * SU) {
        float v[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
          const int t = base + u * NT + tid;
          v[u] = t < n_sub ? sub_max[t] : -INFINITY;
        }
        g(v, base);
      }
    }
  };
  bool spec1_made = false, pair_made = false;
  int spec_blk[4] = {0, 0, 0, 0};  // block-table entries of the first batch's proposals
  const int half = tid >= NT / 2 ? 1 : 0;
  if (kTwoStreams && want0 && want1 && 2 * ahead_blocks<NT>(A.small_batches) <= NT) {
    // both streams at once: the lower half of the workgroup generates the first batch of the base sample,
    // the upper half that of the final sample
    const int blocks0 = ahead_blocks<NT>(A.small_batches, hs, base_draws(hs));
    const int blocks1 = ahead_blocks<NT>(A.small_batches, hs, final_draws(hs));
    const int blocks = half ? blocks1 : blocks0;
    DrawBatch mine = {};
    if (pre_made) {
      // made ahead, while the scores were computed: the proposals are marked as drawn, and the scores of the
      // base sample's proposals are requested
      const uint32_t tk[4] = {pre_t.x, pre_t.y, pre_t.z, pre_t.w};
      uint32_t* tk_bm = half ? taken1 : taken0;
      mine.ok = pre_ok(pre_f);
      mine.first = pre_first(pre_f);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mine.tok[e] = min(max(tk[e], (uint32_t)hs.mid_lo), (uint32_t)max(hs.mid_hi - 1, hs.mid_lo));
        mine.sc[e] = row[mine.tok[e]];
        if ((mine.ok >> e) & 1u) atomicOr(&tk_bm[mine.tok[e] >> 5], 1u << (mine.tok[e] & 31));
      }
      mine.blocks = blocks;
      mine.have_sc = true;
    } else {
      // (selection-only kernel, which runs with every CU full: the scores of the final sample's proposals are
      // requested after the top-k step; a million scattered 4-byte reads at once, from all workgroups in
      // their first microseconds, held every workgroup up for five microseconds at config 3)
      O::make_batch(mine, half ? S1 : S0, hs, 0u, blocks, false, kFused || !half, sm, tid - half * (NT / 2));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) spec_blk[e] = kv_block<kCode>(A.L, seq, (int)mine.tok[e]);
    // (a thread holds draws of one stream; of the other it has the same tokens, none of which counts)
    spec0 = spec1 = mine;
    spec0.ok = half ? 0u : mine.ok;
    spec0.first = half ? 0u : mine.first;
    spec1.ok = half ? mine.ok : 0u;
    spec1.first = half ? mine.first : 0u;
    spec0.blocks = blocks0;
    spec1.blocks = blocks1;
    spec0.have_sc = spec1.have_sc = true;
    spec1_made = true;
    pair_made = true;
  } else if (want0) {
    O::make_batch(spec0, S0, hs, 0u, ahead_blocks<NT>(A.small_batches, hs, base_draws(hs)), false, true, sm, tid);
  } else if (PAIR && PHASE == 1 && kTwoStreams && second && hs.n_s > 0) {
    // (the budget kernel's first batch, which stood in its chain; it depends on the length only)
    DrawBatch mine = {};
    O::make_batch(mine, S1, hs, 0u, budget_blocks<NT>(hs), false, false, sm, tid);
    A.pre_tok[(int64_t)bh * NT + tid] = make_uint4(mine.tok[0], mine.tok[1], mine.tok[2], mine.tok[3]);
    A.pre_flags[(int64_t)bh * NT + tid] = pre_pack(mine, true);
  } else if (second && want1) {
    O::make_batch(spec1, S1, hs, 0u, ahead_blocks<NT>(A.small_batches, hs, final_draws(hs)), false, true, sm, tid);
    spec1_made = true;
  }
  auto clear_cand_hist = [&]() {
    for (int w = tid; w < kBins / 4; w += NT) reinterpret_cast<uint4*>(cand_hist)[w] = make_uint4(0u, 0u, 0u, 0u);
  };
  if (kTwoStreams) clear_cand_hist();  // (make_batch ends with a barrier, and others follow before it is used)
  VATT_STAMP(A.dbg, 1);

  // ---- the head maximum m ----
  float m, lo_sub;  // lo_sub: the smallest maximum of a whole middle sub-tile
  {
    float v_max = -INFINITY, v_min = INFINITY;
    each_sub_batch([&](const float (&v)[SU], int base) {
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const int t = base + u * NT + tid;
        v_max = fmaxf(v_max, v[u]);
        v_min = (t >= sub_lo && t < sub_hi) ? fminf(v_min, v[u]) : v_min;
      }
    });
    v_max = wave_max(v_max);
    v_min = -wave_max(-v_min);
    if ((tid & 63) == 0) {
      ts.wf[0][tid >> 6] = v_max;
      ts.wf[1][tid >> 6] = v_min;
    }
    __syncthreads();
    m = ts.wf[0][0];
    lo_sub = ts.wf[1][0];
#pragma unroll
    for (int w = 1; w < SW; ++w) {
      m = fmaxf(m, ts.wf[0][w]);
      lo_sub = fminf(lo_sub, ts.wf[1][w]);
    }
  }
  S0.m = m;
  S1.m = m;
  VATT_STAMP(A.dbg, 2);

  int topk_flag = 0;
  uint32_t tau_key = 0u;  // largest composite key (~order key: the smallest score) among this thread's top-k members
  float acc_f32 = 0.f;  // this thread's share of D_f = sum over I_f of exp(s_i - m), kept in fp32 per thread
  double acc_f = 0.0;
  bool marked = false;  // the members' weights are in ts.wq, as integers
  uint32_t n_cand_used = 0;  // fast path: members are the candidates marked in bm_f
  constexpr int CPT = kCandCap / NT;  // candidates a thread looks after
  int cand_blk[CPT] = {};
  // (see "more candidates than the list holds")
  uint32_t n_wide_used = 0;
  constexpr uint32_t kWideCap = kCandCap * 12 / sizeof(uint16_t);
  uint16_t* wide = reinterpret_cast<uint16_t*>(cand);
  static_assert(kCapacityMax / kSubTile < 65536, "sub-tiles as 16-bit numbers");
  // f(score, token) for the middle scores of the listed sub-tiles, two lanes per sub-tile, four loads in flight
  auto each_wide = [&](uint32_t count, auto&& f) {
    for (uint32_t q0 = 0; q0 < count; q0 += 4u * (NT / 2)) {
      float4 x[4];
      int tok[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t q = q0 + (uint32_t)(u * (NT / 2) + tid / 2);
        const int t = (int)min((uint32_t)wide[min(q, count - 1)], (uint32_t)(n_sub - 1)) * kSubTile + (tid & 1) * 4;
        x[u] = *reinterpret_cast<const float4*>(row + t);
        tok[u] = q < count ? t : n;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float sv[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (tok[u] + e >= hs.mid_lo && tok[u] + e < hs.mid_hi) f(sv[e], tok[u] + e);
      }
    }
  };
  // ---- I_t (Algorithm 1, top-k step) ----
  {
    const int mid_len = hs.mid_hi - hs.mid_lo;
    if (hs.k > 0) {
      float sT = -INFINITY;
      uint32_t Tidx = kInv32;
      if (hs.k < mid_len) {
        // Fast path.  A lower bound of the k-th largest score: the k-th largest of the sub-tile maxima (of
        // the sub-tiles that lie entirely in the middle region) has at least k middle scores at or above it.
        // Found to one histogram bin, it leaves a few more than k candidates, which are listed in LDS and
        // selected among exactly.
        bool have_T = false;
        if (sub_hi - sub_lo >= hs.k && !A.topk_general) {
          float bound = lo_sub;  // every middle sub-tile maximum is at or above this
          const float scale = (float)(kBins - 1) / (m - lo_sub);
          if (m > lo_sub && scale < 1e30f) {
            each_sub_batch([&](const float (&v)[SU], int base) {
#pragma unroll
              for (int u = 0; u < SU; ++u) {
                const int t = base + u * NT + tid;
                // (no counter for the others: on a short row thousands of additions to one address took 11 K clocks)
                if (t >= sub_lo && t < sub_hi) atomicAdd(&ts.hist[(uint32_t)((m - v[u]) * scale)], 1u);
              }
            });
            __syncthreads();
            TKR::locate_once((uint32_t)hs.k, ts.hist, ts, sm.scan_once[0]);
            // the lower edge of the bin of the k-th largest maximum, a little further down for rounding
            bound = fmaxf(lo_sub, m - ((float)ts.j + 1.02f) / scale);
          }
          VATT_STAMP(A.dbg, 22);
          // sub-tiles that may hold a candidate: those that touch the middle region with a maximum at or
          // above the bound (order in the list does not matter)
          const int sub_first = hs.mid_lo / kSubTile, sub_last = (hs.mid_hi + kSubTile - 1) / kSubTile;
          each_sub_batch([&](const float (&v)[SU], int base) {
            uint64_t mask[SU];
            uint32_t tot = 0;
#pragma unroll
            for (int u = 0; u < SU; ++u) {
              const int t = base + u * NT + tid;
              mask[u] = __ballot(t >= sub_first && t < sub_last && v[u] >= bound);
              tot += (uint32_t)__popcll(mask[u]);
            }
            if (tot) {
              uint32_t at = 0;
              if ((tid & 63) == 0) at = atomicAdd(&ts.qual_n, tot);
              at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
              for (int u = 0; u < SU; ++u) {
                const uint32_t pos = at + lanes_below(mask[u]);
                if (((mask[u] >> (tid & 63)) & 1u) && pos < (uint32_t)kCandCap) qual[pos] = (uint32_t)(base + u * NT + tid);
                at += (uint32_t)__popcll(mask[u]);
              }
            }
          });
          __syncthreads();
          const uint32_t n_qual = ts.qual_n;
          VATT_STAMP(A.dbg, 23);
          VATT_NOTE(A.dbg, 27, n_qual);
          if (n_qual <= (uint32_t)kCandCap) {
            // Candidates: the middle scores of those sub-tiles that are at or above the bound.  Two lanes read the
            // eight scores of a sub-tile; the hits are listed by ballots, one score of every lane at a time (with a
            // prefix sum of the lanes' hits instead, every score was a branch of its own); UQ loads in flight.
            static_assert(kSubTile == 8, "two 16-byte loads per sub-tile");
            const int mid_lo = hs.mid_lo, mid_n = hs.mid_hi - hs.mid_lo;
            auto list_candidates = [&](uint32_t q0, auto uq) {
              constexpr int UQ = decltype(uq)::value;
              float sv[UQ][4];
              int tok[UQ];
#pragma unroll
              for (int u = 0; u < UQ; ++u) {
                const uint32_t q = q0 + (uint32_t)(u * (NT / 2) + tid / 2);
                const int t = (int)min(qual[min(q, n_qual - 1)], (uint32_t)(sub_last - 1)) * kSubTile + (tid & 1) * 4;
                const float4 x = *reinterpret_cast<const float4*>(row + t);
                tok[u] = q < n_qual ? t : n;  // (a token past the row is no middle token)
                sv[u][0] = x.x; sv[u][1] = x.y; sv[u][2] = x.z; sv[u][3] = x.w;
              }
              bool clear = !kTwoStreams && q0 == 0;
              if (q0 == 0 && want1 && !spec1_made) {
                // the final sample's first batch of draws is generated while these loads are in flight
                O::make_batch(spec1, S1, hs, 0u, ahead_blocks<NT>(A.small_batches, hs, final_draws(hs)), false, false, sm, tid);
                spec1_made = true;
                clear = true;
              }
              if (clear) clear_cand_hist();
              auto hits = [&](int u, int e) {
                return __ballot((uint32_t)(tok[u] + e - mid_lo) < (uint32_t)mid_n && sv[u][e] >= bound);
              };
              uint32_t tot = 0;
#pragma unroll
              for (int u = 0; u < UQ; ++u) {
#pragma unroll
                for (int e = 0; e < 4; ++e) tot += (uint32_t)__popcll(hits(u, e));
              }
              if (tot) {
                uint32_t at = 0;
                if ((tid & 63) == 0) at = atomicAdd(&ts.cand_n, tot);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                for (int u = 0; u < UQ; ++u) {
#pragma unroll
                  for (int e = 0; e < 4; ++e) {
                    const uint64_t mask = hits(u, e);
                    const uint32_t pos = at + lanes_below(mask);
                    if (((mask >> (tid & 63)) & 1u) && pos < (uint32_t)kCandCap)
                      cand[pos] = ((uint64_t)(~float_order_key(sv[u][e])) << 32) | (uint32_t)(tok[u] + e);
                    at += (uint32_t)__popcll(mask);
                  }
                }
              }
            };
            if (n_qual <= NT / 2u) list_candidates(0u, std::integral_constant<int, 1>{});
            else
              for (uint32_t q0 = 0; q0 < n_qual; q0 += 4u * (NT / 2)) list_candidates(q0, std::integral_constant<int, 4>{});
            __syncthreads();
          }
          const uint32_t n_cand = n_qual <= (uint32_t)kCandCap ? ts.cand_n : 0u;
          VATT_STAMP(A.dbg, 24);
          VATT_NOTE(A.dbg, 26, n_cand);
          if (n_cand <= (uint32_t)kCandCap && n_cand >= (uint32_t)hs.k) {
            if constexpr (kCode) {
#pragma unroll
              for (int j = 0; j < CPT; ++j) {
                const uint32_t t = (uint32_t)(j * NT + tid);
                if (t < n_cand) cand_blk[j] = kv_block<kCode>(A.L, seq, (int)min((uint32_t)cand[t], (uint32_t)(n - 1)));
              }
            }
            // The members, marked in the bitmap.  (The list order depends on scheduling: the members' weights are
            // summed as 40-bit fixed-point integers, whose sum does not depend on the order; every weight is at most 1.)
            uint64_t fixed_sum = 0;
            auto member = [&](uint64_t c) {
              const uint32_t i = min((uint32_t)c, (uint32_t)(n - 1));
              atomicOr(&bm_f[i >> 5], 1u << (i & 31));
              tau_key = max(tau_key, (uint32_t)(c >> 32));
              fixed_sum += (uint64_t)(__expf(float_from_order_key(~(uint32_t)(c >> 32)) - m) * 1099511627776.0f);
            };
            const float cscale = (float)(kBins - 1) / (m - bound);
            bool by_bin = n_cand > (uint32_t)hs.k && m > bound && cscale < 1e30f;
            uint32_t r = (uint32_t)hs.k;
            auto bin_of = [&](uint64_t c) { return (uint32_t)((m - float_from_order_key(~(uint32_t)(c >> 32))) * cscale); };
            if (by_bin) {
              for (uint32_t t = tid; t < n_cand; t += NT) atomicAdd(&cand_hist[bin_of(cand[t])], 1u);
              __syncthreads();
              VATT_STAMP(A.dbg, 20);
              TKC::locate_once(r, cand_hist, ts, sm.scan_once[1]);
              by_bin = ts.inbin <= (uint32_t)kSmall;
            }
            if (by_bin) {
              // candidates in the bins before rank k's are members; those in its bin are ranked
              const uint32_t j = ts.j;
              r -= ts.below;
              for (uint32_t t = tid; t < n_cand; t += NT) {
                const uint64_t c = cand[t];
                const uint32_t bin = bin_of(c);
                if (bin < j) member(c);
                if (bin == j) ts.slist[min(atomicAdd(&ts.slist_n, 1u), (uint32_t)(kSmall - 1))] = c;
              }
              __syncthreads();
              const uint32_t cnt = min(ts.slist_n, (uint32_t)kSmall);
              if ((uint32_t)tid < cnt) {
                const uint64_t mine = ts.slist[tid];
                uint32_t below = 0;
                for (uint32_t q = 0; q < cnt; ++q) below += (ts.slist[q] < mine) ? 1u : 0u;
                if (below < r) member(mine);
              }
              VATT_STAMP(A.dbg, 21);
            } else {
              CandView<NT> cv;
              cv.list = cand;
              cv.count = n_cand;
              uint64_t T = ~0ull;
              if (n_cand > (uint32_t)hs.k)
                T = TKC::threshold(cv, hs, (uint32_t)hs.k, n_cand, bound, m, scratch, wpre, ts, sm, A.dbg);
              for (uint32_t t = tid; t < n_cand; t += NT)
                if (cand[t] <= T) member(cand[t]);
            }
            fixed_sum = wave_sum(fixed_sum);
            if ((tid & 63) == 0) ts.wq[tid >> 6] = fixed_sum;
            have_T = true;
            marked = true;
            n_cand_used = n_cand;
          }
          if constexpr (NT >= 1024) {
            // More candidates than the list holds (long rows with a large top-k set): the same steps without the list.  Only
            // the sub-tiles are listed, as 16-bit numbers in its place, and their scores are read three times: into the
            // histogram, for the members, and (below) for the ascending list.  Bound by those reads, 100 - 200 KB a pass: with
            // 1 x 128K tokens and k = 3276 the whole selection takes 56 us, with the passes over the whole row that follow
            // below (for a k beyond the number of sub-tiles, or too many scores in one bin) 92 us; whole call 152 -> 116 us.
            const float wscale = (float)(kBins - 1) / (m - bound);
            if (!have_T && n_qual <= kWideCap && m > bound && wscale < 1e30f) {
              __syncthreads();  // the lists and their counters are free
              if (tid == 0) {
                ts.qual_n = 0;
                ts.cand_n = 0;
              }
              clear_cand_hist();
              __syncthreads();
              each_sub_batch([&](const float (&v)[SU], int base) {
                uint64_t mask[SU];
                uint32_t tot = 0;
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                  const int t = base + u * NT + tid;
                  mask[u] = __ballot(t >= sub_first && t < sub_last && v[u] >= bound);
                  tot += (uint32_t)__popcll(mask[u]);
                }
                if (tot) {
                  uint32_t at = 0;
                  if ((tid & 63) == 0) at = atomicAdd(&ts.qual_n, tot);
                  at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                  for (int u = 0; u < SU; ++u) {
                    const uint32_t pos = at + lanes_below(mask[u]);
                    if (((mask[u] >> (tid & 63)) & 1u) && pos < kWideCap) wide[pos] = (uint16_t)(base + u * NT + tid);
                    at += (uint32_t)__popcll(mask[u]);
                  }
                }
              });
              __syncthreads();
              uint32_t mine = 0;
              each_wide(n_qual, [&](float sc, int) {
                if (sc >= bound) {
                  atomicAdd(&cand_hist[(uint32_t)((m - sc) * wscale)], 1u);
                  ++mine;
                }
              });
              mine = wave_sum_u32(mine);
              if ((tid & 63) == 0) atomicAdd(&ts.cand_n, mine);
              __syncthreads();
              TKC::locate_once((uint32_t)hs.k, cand_hist, ts, sm.scan_once[1]);
              if (ts.cand_n >= (uint32_t)hs.k && ts.inbin <= (uint32_t)kSmall) {
                const uint32_t j = ts.j, r = (uint32_t)hs.k - ts.below;
                uint64_t fixed_sum = 0;
                auto member = [&](float sc, uint32_t i) {
                  atomicOr(&bm_f[i >> 5], 1u << (i & 31));
                  tau_key = max(tau_key, ~float_order_key(sc));
                  fixed_sum += (uint64_t)(__expf(sc - m) * 1099511627776.0f);
                };
                each_wide(n_qual, [&](float sc, int i) {
                  const uint32_t bin = (uint32_t)((m - sc) * wscale);
                  if (sc >= bound && bin < j) member(sc, (uint32_t)i);
                  if (sc >= bound && bin == j)
                    ts.slist[min(atomicAdd(&ts.slist_n, 1u), (uint32_t)(kSmall - 1))] = ((uint64_t)(~float_order_key(sc)) << 32) | (uint32_t)i;
                });
                __syncthreads();
                const uint32_t cnt = min(ts.slist_n, (uint32_t)kSmall);
                if ((uint32_t)tid < cnt) {
                  const uint64_t mine_c = ts.slist[tid];
                  uint32_t below = 0;
                  for (uint32_t q = 0; q < cnt; ++q) below += (ts.slist[q] < mine_c) ? 1u : 0u;
                  if (below < r) member(float_from_order_key(~(uint32_t)(mine_c >> 32)), (uint32_t)mine_c);
                }
                fixed_sum = wave_sum(fixed_sum);
                if ((tid & 63) == 0) ts.wq[tid >> 6] = fixed_sum;
                topk_flag = kFlagTopkGeneral;
                have_T = true;
                marked = true;
                n_wide_used = n_qual;
              }
            }
          }
        }
        if (!have_T) {
          topk_flag = kFlagTopkGeneral;
          // General path: histogram over the whole row.  It needs the smallest score of the middle region.
          float v_min = INFINITY, v_max = -INFINITY;
          rv.for_each(hs, [&](float s, int, bool mid) {
            v_min = mid ? fminf(v_min, s) : v_min;
            v_max = mid ? fmaxf(v_max, s) : v_max;
          });
          v_min = -wave_max(-v_min);
          v_max = wave_max(v_max);
          __syncthreads();
          if ((tid & 63) == 0) {
            ts.wf[0][tid >> 6] = v_max;
            ts.wf[1][tid >> 6] = v_min;
          }
          __syncthreads();
          float smax = ts.wf[0][0], smin = ts.wf[1][0];
#pragma unroll
          for (int w = 1; w < SW; ++w) {
            smax = fmaxf(smax, ts.wf[0][w]);
            smin = fminf(smin, ts.wf[1][w]);
          }
          const uint64_t T = TKR::threshold(rv, hs, (uint32_t)hs.k, (uint32_t)mid_len, smin, smax, scratch, wpre, ts,
                                            sm, A.dbg);
          sT = float_from_order_key(~(uint32_t)(T >> 32));
          Tidx = (uint32_t)T;
        }
      }
      VATT_STAMP(A.dbg, 3);
      if (!marked) {
        // Members of the top-k set go into the bitmap: slot u of a wave holds 64 consecutive tokens, so the
        // wave's compare mask is two whole bitmap words, stored by one lane.  A score equal to the threshold
        // score is rare and sends its group through the full comparison.  The weights of the members are
        // added on the way.
        uint64_t* bm64 = reinterpret_cast<uint64_t*>(bm_f);
        rv.for_each_group(hs, [&](const float (&s)[RowView<NT>::kGroup], int i0, auto tag) {
          constexpr int G = RowView<NT>::kGroup;
          constexpr bool kInside = decltype(tag)::value;
          const int first0 = i0 - (tid & 63);  // token of lane 0 in slot 0: a multiple of 64
#pragma unroll
          for (int u = 0; u < G; ++u) {
            const int i = i0 + u * NT;
            const bool mid = kInside || (i >= hs.mid_lo && i < hs.mid_hi);
            const bool take = mid && (s[u] > sT || (s[u] == sT && (uint32_t)i <= Tidx));
            const uint64_t mask = __ballot(take);
            if ((tid & 63) == 0 && (kInside || first0 + u * NT < n)) bm64[(first0 + u * NT) >> 6] = mask;
            if (mask) acc_f32 += take ? __expf(s[u] - m) : 0.f;
            tau_key = take ? max(tau_key, ~float_order_key(s[u])) : tau_key;
          }
        });
      }
      VATT_STAMP(A.dbg, 4);
    }
  }
  VATT_STAMP(A.dbg, 30);
  __syncthreads();
  VATT_STAMP(A.dbg, 31);

  // Fused gather, first part: the V rows (and scores) of this workgroup's share of I_f are requested now and
  // added after the samplers have run.  LPR adjacent lanes read one row; NG rows per round, UF rounds in flight.
  constexpr int LPR = kFused ? FD / 8 : 16;
  constexpr int NG = NT / LPR;
  constexpr int UF = 8;
  const int g_sub = tid % LPR, g_grp = tid / LPR;
  const int kvh = kFused ? div_group(h, A.group) : 0;
  float gacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float gdsum = 0.f;
  uint4 fv[UF];
  float fs[UF];
  int my_nf = 0;
  // contiguous cache: this lane's 8 columns of row 0 of the head's V slice
  const uint16_t* v_head = (kFused && !PAGED)
                               ? A.v + (int64_t)seq * A.L.seq_stride + (int64_t)kvh * A.L.head_stride + g_sub * 8
                               : nullptr;
  // paged cache: the same of the first block; and no code lies beyond the pool
  const uint16_t* v_pool = kCode ? A.v + (int64_t)kvh * A.L.head_stride + g_sub * 8 : nullptr;
  const uint32_t last_code = kCode ? (uint32_t)min(((uint64_t)A.L.num_blocks << A.L.page_shift) - 1u, (uint64_t)kInv32) : 0u;
  auto v_of_code = [&](uint32_t code) {
    const uint32_t in_page = code & ((1u << A.L.page_shift) - 1u);
    return v_pool + (int64_t)(code >> A.L.page_shift) * A.L.block_stride + in_page * (uint32_t)(kFused ? FD : 1);
  };
  // UF rows of a list at once, without branches: all list entries (and their scores) are read from LDS first,
  // then all rows are requested.  The lists are padded to whole calls, so the LDS reads need no bound; a slot
  // beyond the list reads row 0, which add_rows leaves out.  (Written with a per-slot
  // condition, every slot became a branch of its own with an LDS wait inside: sixteen serial LDS round trips.)
  // HaveSc: the scores of the listed tokens are in LDS (list_sc), and the list holds codes (code_of); else (contiguous cache) it holds
  // tokens, and their scores are read from the score row.
  // Rounds beyond the list's end request no rows, in steps of two and four (a round costs the workgroup 128 clocks of
  // address processing and as many of arithmetic, and most lists fill three to five of the eight: 1 x 32K tokens 36.3 -> 35.6 us,
  // one head of 1K 20.1 -> 18.8 us per call).
  // Places [first, count) of a list, as far as a batch reaches, which begins with first's round: place j is always read by lane
  // group j % NG, and a group adds its rows in rising order, so that the sums do not depend on how a list was cut.
  auto round_of = [](int first) { return first & ~(NG - 1); };
  auto load_rows = [&](const uint32_t* list, const float* list_sc, int first, int count, float (&sc)[UF], uint4 (&vv)[UF],
                       auto have_sc) {
    constexpr bool HaveSc = decltype(have_sc)::value;
    uint32_t t[UF];
    const int j0 = round_of(first), jb = j0 + g_grp;
#pragma unroll
    for (int u = 0; u < UF; ++u) {
      t[u] = list[jb + u * NG];
      sc[u] = HaveSc ? list_sc[jb + u * NG] : 0.f;
    }
    static_assert(HaveSc || !kCode, "lists of tokens on a paged cache are walked elsewhere");
#pragma unroll
    for (int u = 0; u < UF; ++u) {
      const bool valid = jb + u * NG >= first && jb + u * NG < count;
      if constexpr (kCode) t[u] = valid ? min(t[u], last_code) : row0_code;
      else t[u] = valid ? min(t[u], (uint32_t)(n - 1)) : 0u;
    }
    auto rows = [&](auto from, auto to) {
#pragma unroll
      for (int u = decltype(from)::value; u < decltype(to)::value; ++u) {
        if constexpr (!HaveSc) sc[u] = row[t[u]];
        if constexpr (kCode) {
          vv[u] = load_stream_16(v_of_code(t[u]));
        } else {
          vv[u] = load_stream_16(v_head + t[u] * (uint32_t)(kFused ? FD : 1));  // (n_max * d < 2^32)
        }
      }
    };
    rows(Int<0>{}, Int<2>{});
    if (count > j0 + 2 * NG) rows(Int<2>{}, Int<4>{});
    if (count > j0 + 4 * NG) rows(Int<4>{}, Int<UF>{});
  };
  // entries of this workgroup's share of the first c places of the final sample
  auto share_of = [&](uint32_t c) { return c > split ? (int)((c - split + smask) >> shift) : 0; };
  using ScInLds = std::true_type;
  using ScInRow = std::false_type;
  if constexpr (kFused) my_nf = (int)(g_hi - g_lo);

  VATT_STAMP(A.dbg, 32);
  if (!(PAIR && PHASE == 1) && want1 && !spec1_made) O::make_batch(spec1, S1, hs, 0u, ahead_blocks<NT>(A.small_batches, hs, final_draws(hs)), false, false, sm, tid);

  // ---- I_bs (Algorithm 2, base sample) and the sums over it ----
  int flags = topk_flag;
  double acc_w = 0.0, acc_w2 = 0.0;
  // Usual case (both first batches at hand, base sample neither the whole residual nor taken as a
  // complement): the draws of both streams are tested against the top-k set and counted in draw order by ONE
  // workgroup scan (the lower half of the workgroup holds the base sample's stream, the upper half the final
  // sample's; the two counts travel in the halves of one word), which also counts the top-k bitmap's bits.  The base
  // sample is complete if its first batch holds b0 accepted draws.  And since the budget is never below b0, the first b0
  // accepted draws of the other stream belong to the final sample whatever the budget turns out to be (unless it asks for
  // so much that the sample is taken as a complement): with the fused gather their V rows are requested now, and are in
  // when the budget is known.  From the marked members to the budget there are four barriers where the lists, the sums and the
  // samples, one after the other, had ten: a barrier with the scan or the sums around it is 300 - 400 clocks of the chain (1 x
  // 32K tokens 35.6 -> 35.0 us, one head of 1K 18.8 -> 17.7 us per call).  (The sorted and the nested forms of the lists are made
  // by the general path only.)
  // The lists of I_f, once wpre is complete (and, with the fused gather, this workgroup's share of them in LDS).
  auto write_lists = [&]() {
    // ascending list of the top-k tokens
    if (hs.k > 0) {
      if (NT >= 1024 && n_wide_used) {
        each_wide(n_wide_used, [&](float sc, int i) {
          const uint32_t word = bm_f[i >> 5], bit = 1u << (i & 31);
          if (word & bit) {
            const uint32_t pos = wpre[i >> 5] + (uint32_t)__popc(word & (bit - 1u));
            if (pos < (uint32_t)A.k_max) {
              idx[A.seg_topk + pos] = i;
              place_sc[A.seg_topk + pos] = sc;
            }
          }
        });
      } else if (marked) {
        // every member sits in the candidate list: its place in the ascending list is the number of members
        // below it, from the word prefix and the bits below its own (no thread walks a crowded word)
        auto place_member = [&](uint32_t t, int blk) {
          const uint64_t c = cand[t];
          const uint32_t i = min((uint32_t)c, (uint32_t)(n - 1));
          const uint32_t word = bm_f[i >> 5], bit = 1u << (i & 31);
          if (word & bit) {
            const uint32_t pos = wpre[i >> 5] + (uint32_t)__popc(word & (bit - 1u));
            if ((kFused ? writer : lister) && pos < (uint32_t)A.k_max) idx[A.seg_topk + pos] = (int32_t)i;
            if (!kFused && pos < (uint32_t)A.k_max) place_sc[A.seg_topk + pos] = float_from_order_key(~(uint32_t)(c >> 32));
            to_glist((uint32_t)(hs.n_sink + hs.n_win) + pos, code_of(i, blk), float_from_order_key(~(uint32_t)(c >> 32)));
          }
        };
        if constexpr (kCode) {
#pragma unroll
          for (int j = 0; j < CPT; ++j)
            if ((uint32_t)(j * NT + tid) < n_cand_used) place_member((uint32_t)(j * NT + tid), cand_blk[j]);
        } else {
          for (uint32_t t = tid; t < n_cand_used; t += NT) place_member(t, 0);
        }
      } else {
        const int wpt = (words + NT - 1) / NT;
        const int w0 = tid * wpt;
        for (int w = w0; w < min(w0 + wpt, words); ++w) {
          uint32_t bits = bm_f[w];
          uint32_t pos = wpre[w];
          while (bits) {
            const int i = (w << 5) + (__ffs(bits) - 1);
            bits &= bits - 1u;
            if ((kFused ? writer : lister) && pos < (uint32_t)A.k_max) idx[A.seg_topk + pos] = i;
            if (kFused) to_glist((uint32_t)(hs.n_sink + hs.n_win) + pos, row_code((uint32_t)i), row[i]);
            else if (pos < (uint32_t)A.k_max) place_sc[A.seg_topk + pos] = row[i];
            ++pos;
          }
        }
      }
    }
    for (int i = tid; i < hs.n_sink; i += NT) {
      if (kFused ? writer : lister) idx[A.seg_sink + i] = i;
      if (kFused) to_glist((uint32_t)i, i == tid ? code_of((uint32_t)i, edge0_blk) : row_code((uint32_t)i), i == tid ? edge0 : row[i]);
      else place_sc[A.seg_sink + i] = i == tid ? edge0 : row[i];
    }
    for (int i = tid; i < hs.n_win; i += NT) {
      if (kFused ? writer : lister) idx[A.seg_win + i] = hs.mid_hi + i;
      if (kFused) {
        const uint32_t tok = (uint32_t)(hs.mid_hi + i);
        to_glist((uint32_t)(hs.n_sink + i), i == tid ? code_of(tok, edge1_blk) : row_code(tok), i == tid ? edge1 : row[tok]);
      }
      else place_sc[A.seg_win + i] = i == tid ? edge1 : row[hs.mid_hi + i];
    }
  };
  bool fast_base = false, spec_dyn = false;
  uint32_t acc_bits = 0, acc_pos = 0, tot1 = 0;
  float dacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // final-sample rows, before the factor n_s / b
  float ddsum = 0.f;
  uint4 dv[UF];
  float ds[UF];
  int my_spec = 0;
  // A further batch of rows under way: the second of I_f, or what the first draws add to a final sample beyond the base sample's
  // size (2 x 20K tokens with budgets up to 2276: 45.6 -> 44.3 us per call; 8 x 0.5K - 7K, whose lists have two batches, 35.1 ->
  // 34.4).  It takes 40 registers more, which 512 threads have.
  uint4 ev[UF];
  float es[UF];
  {
    const uint32_t ns = (uint32_t)hs.n_s, c0 = (uint32_t)hs.b0;
    const bool usual = kTwoStreams && PHASE == 0 && (kFused || (!A.ascending && !A.nested)) && pair_made && hs.n_s > 0 &&
                       c0 < ns && 2u * c0 <= ns;
    const bool listed = hs.k > 0;
    auto test_draws = [&]() {
      const DrawBatch& B = half ? spec1 : spec0;
      acc_bits = B.first & ~O::test_bits4(bm_f, B.tok);
      return (uint32_t)__popc(acc_bits) << (half ? 16 : 0);
    };
    uint32_t taken = 0, total = 0;
    if constexpr (kFused) {
      const int wpt = (words + NT - 1) / NT, w0 = tid * wpt;
      uint32_t bits = 0;
      if (listed)
        for (int w = w0; w < min(w0 + wpt, words); ++w) bits += __popc(bm_f[w]);
      if (usual) taken = test_draws();
      block_exclusive_scan_two_once<NT>(bits, taken, &total, sm.scan_once[2], sm.scan_once[3]);
      if (listed) {
        for (int w = w0; w < min(w0 + wpt, words); ++w) {
          wpre[w] = bits;
          bits += __popc(bm_f[w]);
        }
      }
    } else {
      // (the lists leave, and the final sample's scores are asked for, as early as they can: with every CU full this
      // kernel is bound by its scattered reads, and the gather kernel behind it takes 3 us longer when they come late)
      if (lister) {
        if (listed) O::word_prefix(bm_f, words, wpre, sm, &sm.scan_once[2]);
        write_lists();
      }
      if (second) {
        const uint32_t acc = spec1.first & ~O::test_bits4(bm_f, spec1.tok);
        uint32_t unused, pos = block_exclusive_scan_once<NT>((uint32_t)__popc(acc), &unused, sm.scan_once[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool a = (acc >> e) & 1u;
          if (a && pos < (uint32_t)A.b_max) place_sc[A.seg_dyn + pos] = spec1.sc[e];
          pos += a ? 1u : 0u;
        }
        return;
      }
      if (pair_made && half) {  // (whole waves: the upper half holds the final sample's proposals)
#pragma unroll
        for (int e = 0; e < 4; ++e) spec0.sc[e] = spec1.sc[e] = row[spec1.tok[e]];
      }
      if (usual) taken = block_exclusive_scan_once<NT>(test_draws(), &total, sm.scan_once[3]);
    }
    if (usual) {
      tot1 = total >> 16;
      acc_pos = half ? taken >> 16 : taken & 0xffffu;
      fast_base = (total & 0xffffu) >= c0;
      spec_dyn = fast_base && tot1 >= c0;
    }
    if (fast_base) {
      uint32_t pos = acc_pos;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool a = (acc_bits >> e) & 1u;
        const bool take = a && pos < (uint32_t)hs.b0;
        if (!half) {
          if (take && writer && pos < (uint32_t)A.b0_max) idx[A.seg_base + pos] = (int32_t)spec0.tok[e];
          const double w = take ? (double)__expf(spec0.sc[e] - m) : 0.0;
          acc_w += w;
          acc_w2 += w * w;
        } else if (kFused && spec_dyn && take && (pos & smask) == split && (pos >> shift) < (uint32_t)A.dlist_cap) {
          dlist[pos >> shift] = code_of(spec1.tok[e], spec_blk[e]);
          dlist_sc[pos >> shift] = spec1.sc[e];
        }
        pos += a ? 1u : 0u;
      }
    }
  }
  // weights of the sink and window tokens (their scores were requested at the start)
  acc_f32 += __expf(edge0 - m) + __expf(edge1 - m);  // exp(-inf) = 0 for threads without a token
  for (int i = tid + NT; i < hs.n_sink; i += NT) acc_f32 += __expf(row[i] - m);
  for (int i = tid + NT; i < hs.n_win; i += NT) acc_f32 += __expf(row[hs.mid_hi + i] - m);
  if (tid == NT - kWave && marked) {
    uint64_t tot = 0;
#pragma unroll
    for (int w = 0; w < SW; ++w) tot += ts.wq[w];
    acc_f += (double)tot * (1.0 / 1099511627776.0);
  }
  acc_f += (double)acc_f32;
  double sums[3] = {acc_f, acc_w, acc_w2};
  const bool posted = fast_base || hs.n_s == 0;  // the sums are complete
  if (posted) O::block_sum_post(sums, sm);
  __syncthreads();
  VATT_STAMP(A.dbg, 5);
  if constexpr (kFused) {
    if (spec_dyn) {
      my_spec = min(share_of((uint32_t)hs.b0), A.dlist_cap);
      load_rows(dlist, dlist_sc, 0, my_spec, ds, dv, ScInLds{});
    }
  }
  if constexpr (kFused) {
    write_lists();
    __syncthreads();
    load_rows(glist, glist_sc, 0, my_nf, fs, fv, ScInLds{});
    if (my_nf > UF * NG) load_rows(glist, glist_sc, UF * NG, my_nf, es, ev, ScInLds{});
  }
  if (hs.n_s > 0 && !fast_base) {
    Emit E0 = emit_to(idx + A.seg_base, (uint32_t)A.b0_max);
    E0.global = writer;
    const int f = O::draw_sample(S0, hs, (uint32_t)hs.b0, spec0, want0, A.small_batches, E0, &acc_w, &acc_w2, sm);
    flags |= ((f & 1) ? kFlagBaseComplement : 0) | ((f & 2) ? kFlagBaseBatches : 0) | ((f & 4) ? kFlagDrawCap : 0);
    if (A.ascending && !(f & 1))
      O::sort_ascending(idx + A.seg_base, (uint32_t)min(hs.b0, A.b0_max), scratch, wpre, n, sm);
    VATT_STAMP(A.dbg, 5);
  }
  if constexpr (PHASE == 1) {
    if (tid == 0) {
      HeadRec r;
      r.m = m;
      r.scale = 0.f;
      r.n = n;
      r.n_sink = hs.n_sink;
      r.n_win = hs.n_win;
      r.k = hs.k;
      r.b = hs.n_s > 0 ? hs.b0 : 0;  // the statistics pass walks the base sample
      r.n_s = hs.n_s;
      r.b_keep = 0;
      r.base_cached = 0;
      r.tail_by_token = 1;  // (the statistics pass walks the base sample, whose scores are not at its places)
      A.head_rec[bh] = r;
      A.out_counts[(int64_t)bh * 8 + 7] = flags;
    }
    return;
  }

  // ---- statistics (Algorithm 2, get-stats): w_i = exp(s_i - m) ----
  // For the range-based Hoeffding budget: every residual token scores at most the weakest top-k member, so the
  // residual weights lie in [0, exp(min_{I_t} s - m)]; without a top-k set only w <= 1 is known.
  double w_range = 1.0;
  if (A.range_factor > 0.0 && hs.k > 0) {
    const uint32_t wk = wave_max_u32(tau_key);
    if ((tid & 63) == 0) ts.wu[0][tid >> 6] = wk;
    __syncthreads();
    uint32_t key = 0u;
#pragma unroll
    for (int w = 0; w < SW; ++w) key = max(key, ts.wu[0][w]);
    w_range = exp((double)float_from_order_key(~key) - (double)m);
  }
  // Long rows (1024 threads; their samples hold thousands of tokens and the first batch of draws usually holds
  // the whole final sample): the scores of that batch's proposals are requested now and arrive under the sums
  // and the budget; they go to the list places with the accepted tokens.  (In the 512-thread kernel, which is
  // short of registers, the same cost more than the gather gains: a sample that its shortcut above does not
  // cover is read by token.)
  constexpr bool kEmitScores = !kFused && NT >= 1024;
  if (kEmitScores && !PAIR && want1 && !spec1.have_sc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) spec1.sc[e] = row[min(spec1.tok[e], (uint32_t)(n - 1))];
    spec1.have_sc = true;
  }
  if (!posted) {
    sums[1] = acc_w;
    sums[2] = acc_w2;
    O::block_sum_post(sums, sm);
    __syncthreads();
  }
  O::block_sum_get(sums, sm);
  VATT_STAMP(A.dbg, 6);
  const double D_f = sums[0];
  double b_star = 0.0;
  int bfin = 0;
  int n_s = hs.n_s;
  asm("" : "+s"(n_s));  // (worked out anew: its double, which the sizes at the start need too, was kept to the end and spilled)
  if (n_s > 0) {
    const Budget bud = algorithm2_budget(A, n_s, hs.b0, D_f, sums[1], sums[2], 0.0, w_range);
    b_star = bud.b_star;
    bfin = bud.b;
    const double D_hat = bud.D_hat;
    if (tid == 0 && writer && A.out_stats) {
      float* st = A.out_stats + (int64_t)bh * 4;
      st[0] = (float)D_hat;
      st[1] = (float)bud.sigma2;
      st[2] = st[3] = 0.f;
    }
  } else if (tid == 0 && writer && A.out_stats) {
    float* st = A.out_stats + (int64_t)bh * 4;
    st[0] = (float)D_f;
    st[1] = st[2] = st[3] = 0.f;
  }

  VATT_STAMP(A.dbg, 7);
  // ---- I_dyn (Algorithm 1, final sample) ----
  bool fast_dyn = false, more_dyn = false;
  int j_coded = 0, j_done = 0;  // fused gather: places of the share that hold codes and scores; that are requested
  {
    // the first batch of draws holds the whole final sample, and it is not taken as a complement: its members
    // are the accepted draws counted above, up to the budget
    fast_dyn = spec_dyn && (uint32_t)bfin <= tot1 && 2u * (uint32_t)bfin <= (uint32_t)hs.n_s;
    // the same draws begin a larger sample: fused gather, all of them are listed with their scores, and the first rows the list
    // has beyond those of the base sample's size are requested before the further draws are made
    more_dyn = kFused && spec_dyn && !fast_dyn && 2u * (uint32_t)bfin <= (uint32_t)hs.n_s;
    if (fast_dyn || more_dyn) {
      uint32_t pos = acc_pos;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool a = (acc_bits >> e) & 1u;
        if (half && a && pos < (uint32_t)bfin) {
          if (writer && pos < (uint32_t)A.b_max) idx[A.seg_dyn + pos] = (int32_t)spec1.tok[e];
          if (!kFused && pos < (uint32_t)A.b_max) place_sc[A.seg_dyn + pos] = spec1.sc[e];
          if (kFused && pos >= (uint32_t)hs.b0 && (pos & smask) == split && (pos >> shift) < (uint32_t)A.dlist_cap) {
            dlist[pos >> shift] = code_of(spec1.tok[e], spec_blk[e]);
            dlist_sc[pos >> shift] = spec1.sc[e];
          }
        }
        pos += a ? 1u : 0u;
      }
      if constexpr (kFused) {
        __syncthreads();
        j_coded = min(share_of((uint32_t)min((uint32_t)bfin, tot1)), A.dlist_cap);
        j_done = min(UF * NG, my_spec);
        if (my_nf <= UF * NG && j_coded > j_done) {
          load_rows(dlist, dlist_sc, j_done, j_coded, es, ev, ScInLds{});
        }
      }
    }
  }
  bool dyn_placed = fast_dyn;  // the final sample's scores are at its list places
  if (bfin > 0 && !fast_dyn) {
    Emit E1 = emit_to(idx + A.seg_dyn, (uint32_t)A.b_max);
    E1.global = writer;
    if (kEmitScores) E1.sc_dst = place_sc + A.seg_dyn;
    if (kFused) {
      E1.lds = dlist;
      E1.lds_cap = (uint32_t)A.dlist_cap;
      E1.shift = shift;
      E1.split = split;
    }
    const int f = (!kFused && A.nested)
                      ? O::draw_nested(S1, hs, (uint32_t)hs.b0, (uint32_t)bfin, bm_f, idx + A.seg_base,
                                       idx + A.seg_dyn, (uint32_t)A.b_max, A.small_batches, sm)
                      : O::draw_sample(S1, hs, (uint32_t)bfin, spec1, want1 && !more_dyn, A.small_batches, E1, nullptr, nullptr, sm,
                                       more_dyn ? tot1 : 0u, more_dyn ? (uint32_t)spec1.blocks : 0u);
    flags |= ((f & 1) ? kFlagDynComplement : 0) | ((f & 2) ? kFlagDynBatches : 0) | ((f & 4) ? kFlagDrawCap : 0);
    // (one batch made ahead with its scores held the whole sample, and the list stays in acceptance order)
    dyn_placed = kEmitScores && !A.nested && !A.ascending && want1 && (spec1.have_sc || PAIR) && f == 0;
    if (!kFused && A.ascending && !A.nested && !(f & 1))
      O::sort_ascending(idx + A.seg_dyn, (uint32_t)min(bfin, A.b_max), scratch, wpre, n, sm);
    VATT_STAMP(A.dbg, 8);
  }
  if (tid == 0 && writer) {
    int32_t* c = A.out_counts + (int64_t)bh * 8;
    c[0] = hs.n_sink;
    c[1] = hs.n_win;
    c[2] = hs.k;
    c[3] = hs.n_s > 0 ? hs.b0 : 0;
    c[4] = bfin;
    c[5] = hs.n_s;
    c[6] = n;
    c[7] = flags;
    if (A.out_budget_raw) A.out_budget_raw[bh] = b_star;
    HeadRec r;
    r.m = m;
    r.scale = bfin > 0 ? (float)((double)n_s / (double)bfin) : 0.f;
    r.n = n;
    r.n_sink = hs.n_sink;
    r.n_win = hs.n_win;
    r.k = hs.k;
    r.b = bfin;
    r.n_s = hs.n_s;
    r.b_keep = (A.nested && bfin > 0) ? hs.b0 : 0;
    r.base_cached = 0;
    r.tail_by_token = dyn_placed ? 0 : 1;
    A.head_rec[bh] = r;
  }
  VATT_STAMP(A.dbg, 9);

  // Fused gather, second part: add the rows of I_f that were requested above, then the rest of I_f (only long
  // lists have one), then this workgroup's share of the final sample with the weight factor n_s / b.
  if constexpr (kFused) {
    // A slot beyond the list adds nothing: with weight 0 the Inf of a row that is not listed would make a NaN.  A whole batch has no
    // such slots and tests none (8 x 7K tokens with lists of 3400 rows 65.3 us per call, with the tests 70.5).
    auto add_one = [&](float (&acc)[8], float& dsum, float sc, const uint4& vv) {
      const float wt = __expf(sc - m);
      add_weighted_row(acc, wt, vv);
      dsum += g_sub == 0 ? wt : 0.f;
    };
    // (the rounds that load_rows requested for the same places)
    auto add_rows = [&](float (&acc)[8], float& dsum, const float (&sc)[UF], const uint4 (&vv)[UF], int first, int count) {
      const int j0 = round_of(first);
      if (j0 == first && count >= j0 + UF * NG) {
#pragma unroll
        for (int u = 0; u < UF; ++u) add_one(acc, dsum, sc[u], vv[u]);
        return;
      }
      auto part = [&](auto from, auto to) {
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(to)::value; ++u)
          if ((uint32_t)(j0 - first + u * NG + g_grp) < (uint32_t)(count - first)) add_one(acc, dsum, sc[u], vv[u]);
      };
      part(Int<0>{}, Int<2>{});
      if (count > j0 + 2 * NG) part(Int<2>{}, Int<4>{});
      if (count > j0 + 4 * NG) part(Int<4>{}, Int<UF>{});
    };
    // the rest of a list from place j0 on: a batch of rows is requested before the one in front of it is added
    auto rest = [&](float (&acc)[8], float& dsum, const uint32_t* list, const float* list_sc, int j0, int count, auto have_sc) {
      if (j0 >= count) return;
      load_rows(list, list_sc, j0, count, fs, fv, have_sc);
      for (;;) {
        const int j1 = round_of(j0) + UF * NG, j2 = j1 + UF * NG;
        if (j1 < count) load_rows(list, list_sc, j1, count, es, ev, have_sc);
        add_rows(acc, dsum, fs, fv, j0, count);
        if (j1 >= count) break;
        if (j2 < count) load_rows(list, list_sc, j2, count, fs, fv, have_sc);
        add_rows(acc, dsum, es, ev, j1, count);
        if (j2 >= count) break;
        j0 = j2;
      }
    };
    if (my_nf > 0) add_rows(gacc, gdsum, fs, fv, 0, my_nf);
    if (my_nf > UF * NG) {
      add_rows(gacc, gdsum, es, ev, UF * NG, my_nf);
      rest(gacc, gdsum, glist, glist_sc, 2 * UF * NG, my_nf, ScInLds{});
    }
    static_assert((NG & (NG - 1)) == 0, "round_of");
    const int my_nd = min(share_of((uint32_t)bfin), A.dlist_cap);
    if (fast_dyn || more_dyn) {
      if (my_spec > 0) add_rows(dacc, ddsum, ds, dv, 0, my_spec);
      if (my_nf <= UF * NG && j_coded > j_done) {
        add_rows(dacc, ddsum, es, ev, j_done, j_coded);
        j_done = min(round_of(j_done) + UF * NG, j_coded);
      }
      rest(dacc, ddsum, dlist, dlist_sc, j_done, j_coded, ScInLds{});
    }
    // What further draws or a complement left is listed by token.  On a paged cache its rows wait for their block-table entries: a batch
    // at a time, loads and sums in one piece of code (read a batch ahead in parts, as by rest, every part's sums wait for the rows
    // just requested: 8 x 0.5K - 7K tokens with whole residuals 91 -> 81 us per call, 8 x 9K 133 -> 121; on a contiguous cache, whose
    // rows wait for nothing else, a batch ahead is better, 67 us against 72).
    if constexpr (kCode) {
      int j0 = j_coded;
      auto batch = [&](auto whole) {
        constexpr bool Whole = decltype(whole)::value;
        const int jb = round_of(j0) + g_grp;
        auto listed = [&](int u) { return Whole || (uint32_t)(jb + u * NG - j0) < (uint32_t)(my_nd - j0); };
        uint32_t t[UF];
        int blk[UF];
#pragma unroll
        for (int u = 0; u < UF; ++u) t[u] = dlist[jb + u * NG];
#pragma unroll
        for (int u = 0; u < UF; ++u) {
          t[u] = listed(u) ? min(t[u], (uint32_t)(n - 1)) : 0u;
          blk[u] = kv_block<true>(A.L, seq, (int)t[u]);
        }
#pragma unroll
        for (int u = 0; u < UF; ++u) {
          fs[u] = row[t[u]];
          fv[u] = load_stream_16(v_of_code(code_of(t[u], blk[u])));
        }
#pragma unroll
        for (int u = 0; u < UF; ++u)
          if (listed(u)) add_one(dacc, ddsum, fs[u], fv[u]);
      };
      if (j0 < my_nd && round_of(j0) != j0) {  // behind the places that hold codes
        batch(std::false_type{});
        j0 = round_of(j0) + UF * NG;
      }
      for (; j0 + UF * NG <= my_nd; j0 += UF * NG) batch(std::true_type{});
      if (j0 < my_nd) batch(std::false_type{});
    } else {
      rest(dacc, ddsum, dlist, dlist_sc, j_coded, my_nd, ScInRow{});
    }
    const float tail_scale = bfin > 0 ? (float)((double)hs.n_s / (double)bfin) : 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) gacc[c] += tail_scale * dacc[c];
    gdsum += tail_scale * ddsum;
    VATT_STAMP(A.dbg, 10);
    // lane groups of a wave hold different rows: add them, then the waves through LDS
    const int lane = tid & 63, wave = tid >> 6;
    add_lane_groups<LPR>(gacc);
    gdsum = wave_sum_f32(gdsum);
    float* g_d = g_red + SW * FD;
    if (LPR == 16 || (lane & 8) == 0) {
      const int col = lane_groups_column<LPR>(lane);
      g_red[wave * FD + col] = gacc[0];
      g_red[wave * FD + col + 1] = gacc[1];
    }
    if (lane == 0) g_d[wave] = gdsum;
    __syncthreads();
    float dtot = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < SW; ++w2) dtot += g_d[w2];
    float* part = A.part + ((int64_t)bh * A.splits + split) * (FD + 4);
    if (tid < FD) {
      float a = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < SW; ++w2) a += g_red[w2 * FD + tid];
      if (ALONE) A.out_o[(int64_t)bh * FD + tid] = a / dtot;
      else part[tid] = a;
    }
    if (tid == 0) {
      if (!ALONE) part[FD] = dtot;
      else if (A.out_lse) A.out_lse[bh] = m + logf(dtot);
    }
    VATT_STAMP(A.dbg, 11);
  }
}

typedef void (*HeadKernel)(HeadArgs);
// The instantiation for a plan: workgroup size; with the fused gather also head dimension and cache layout.
template <int D, bool PAGED>
HeadKernel fused_kernel_for(bool alone, bool options) {
  if (alone) return options ? head_kernel<kHeadThreads, D, PAGED, true, 0, true, false> : head_kernel<kHeadThreads, D, PAGED, true, 0, false, false>;
  return options ? head_kernel<kHeadThreads, D, PAGED, false, 0, true, false> : head_kernel<kHeadThreads, D, PAGED, false, 0, false, false>;
}
HeadKernel fused_kernel_for(int d, bool paged, bool alone, bool options) {
  if (d == 128) return paged ? fused_kernel_for<128, true>(alone, options) : fused_kernel_for<128, false>(alone, options);
  return paged ? fused_kernel_for<64, true>(alone, options) : fused_kernel_for<64, false>(alone, options);
}
template <int NT, bool OPTIONS>
HeadKernel head_kernel_for(int phase) {
  return phase == 0 ? head_kernel<NT, 0, false, false, 0, OPTIONS, false> : head_kernel<NT, 0, false, false, 1, OPTIONS, false>;
}
// pair: as head_pair says (never with options, nor for phase 0 with 512 threads)
HeadKernel head_kernel_for(int threads, int phase, bool options, bool pair) {
  if (pair && threads == kHeadThreadsLong)
    return phase == 0 ? head_kernel<kHeadThreadsLong, 0, false, false, 0, false, true> : head_kernel<kHeadThreadsLong, 0, false, false, 1, false, true>;
  if (pair) return head_kernel<kHeadThreads, 0, false, false, 1, false, true>;
  if (threads == kHeadThreadsLong) return options ? head_kernel_for<kHeadThreadsLong, true>(phase) : head_kernel_for<kHeadThreadsLong, false>(phase);
  return options ? head_kernel_for<kHeadThreads, true>(phase) : head_kernel_for<kHeadThreads, false>(phase);
}

}  // namespace

hipError_t set_kernel_attributes(const Plan& pl) {
  // The limit on dynamic LDS belongs to the kernel, not to the plan: it is raised to all a CU has (less the
  // kernels' static part), so that plans of different capacities can be used in any order.
  const int cap = 160 * 1024 - (int)head_kernel_static_lds_bytes();
  auto raise = [&](HeadKernel f) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, cap);
  };
  for (const int threads : {kHeadThreads, kHeadThreadsLong})
    for (const int phase : {0, 1})
      for (const bool options : {false, true}) {
        const hipError_t e = raise(head_kernel_for(threads, phase, options, false));
        if (e != hipSuccess) return e;
        if (options || (threads == kHeadThreads && phase == 0)) continue;
        const hipError_t e2 = raise(head_kernel_for(threads, phase, false, true));
        if (e2 != hipSuccess) return e2;
      }
  for (const int d : {64, 128})
    for (const bool paged : {false, true})
      for (const bool alone : {false, true})
        for (const bool options : {false, true}) {
          const hipError_t e = raise(fused_kernel_for(d, paged, alone, options));
          if (e != hipSuccess) return e;
        }
  const hipError_t e = set_budget_kernel_attributes();
  return e != hipSuccess ? e : set_given_kernel_attributes(pl);
}

size_t head_kernel_lds_bytes(int n_max, int head_threads) {
  return sizeof(uint32_t) * (head_threads == kHeadThreadsLong ? head_lds<kHeadThreadsLong, false>(n_max) : head_lds<kHeadThreads, true>(n_max)).lists;
}

// LDS entries of a workgroup's share of I_f and of the final sample when `splits` workgroups share a head.
// (padded to whole calls of the row loader: 8 rounds of NT / (d / 8) rows, 512 entries at d = 64,
// and one call more, since the final sample's list is also walked from a start that is not a multiple of a call)
int fused_glist_cap(const Plan& pl, int splits) { return ((pl.p.sink + pl.p.window + pl.k_max) / splits + 2 + 1023) & ~511; }
int fused_dlist_cap(const Plan& pl, int splits) { return (pl.b_max / splits + 2 + 1023) & ~511; }
// Dynamic LDS of the selection kernel with the fused gather (512 threads).
size_t fused_head_lds_bytes(const Plan& pl, int splits) {
  return head_kernel_lds_bytes(pl.p.n_max, kHeadThreads) +
         ((size_t)fused_glist_cap(pl, splits) + (size_t)fused_dlist_cap(pl, splits)) * (sizeof(uint32_t) + sizeof(float)) +
         (size_t)(kHeadThreads / kWave) * (pl.p.head_dim + 1) * sizeof(float) + 64;
}

size_t head_kernel_static_lds_bytes() { return sizeof(TopkSmem) + 64; }

hipError_t launch_head(const Plan& pl, int phase, const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws,
                       int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                       hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  const vatt_params& p = pl.p;
  const bool pair = head_pair(pl, phase);
  A.splits = pair ? 2 : 1;
  if (phase == 1) {  // (from its second workgroups to the budget kernel)
    A.pre_tok = reinterpret_cast<uint4*>(static_cast<char*>(ws) + pl.off_pre_tok);
    A.pre_flags = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pl.off_pre_flags);
  }
  hipLaunchKernelGGL(head_kernel_for(pl.head_threads, phase, head_options(pl), pair), dim3(p.n_q_heads, pl.vbatch, A.splits), dim3(pl.head_threads), pl.head_lds_bytes, st, A);
  return hipGetLastError();
}

bool fused_splits_fit(const Plan& pl, int splits) {
  if (splits < 1 || splits > 16 || (splits & (splits - 1)) != 0) return false;
  if (pl.head_threads != kHeadThreads || pl.p.target != VATT_TARGET_D) return false;
  return fused_head_lds_bytes(pl, splits) + head_kernel_static_lds_bytes() <= 160 * 1024;
}

// Workgroups per head of the fused kernel, all of them at once on the chip, one per compute unit; 0: separate kernels.
// With one per head the merge launch falls away, which is worth two to three microseconds as long as its lists are short.
// Measured (whole call, us, separate kernels or the largest power of two that fits -> one per head; with the count of
// workgroups a constant of the kernel, as it is now, another 0.6 to 1.5 less):
//   more heads than half the compute units, 256 heads of 300 / 4K / 7K paged / 9K tokens: 34.7 -> 33.0, 39.8 -> 36.0, 41.5 -> 39.8,
//     55.7 -> 51.3, none left at 12K (where the list of a final sample as long as the row no longer fits); multi-query steps,
//     whose first draws are not made beside the scores, gain from about 200 heads on (8 query tokens, 4K: 40.1 -> 38.2, 5: 35.5 -> 37.0);
//   fewer heads: one head of 1K 23.7 -> 21.7, 32 heads of 4K / 9K 27.5 -> 25.4, 28.2 -> 27.0, but 32 heads of 9K with a list of 1156
//     rows 30.2 -> 30.8, of 12K (856 rows) 30.8 -> 31.2, with 4 query tokens of 2K 34.2 -> 35.3.
// That is with budgets at the base sample's size.  They grow with (z / epsilon)^2, and one workgroup then gathers all of a
// long list: 32 heads of 8K at epsilon 0.05 / 0.03 / 0.02 / 0.01 with eight per head 26.5 / 28.8 / 32.6 / 38.2, with one 24.8 /
// 31.6 / 40.5 / 60.9, of 2K 25.2 / 27.7 / 28.9 / 28.3 and 23.2 / 27.6 / 32.6 / 31.4, of 1K 24.7 / 28.6 / 28.2 / 28.0 and 22.5 / 27.0 / 27.3 /
// 27.3; so a tight epsilon (0.035 at delta 0.05) takes one workgroup only for few heads' short rows.  256 heads of 7K at 0.02 /
// 0.01: apart 53.4 / 60.9, one per head 50.4 / 65.9.
int fused_splits_for(const Plan& pl) {
  const vatt_params& p = pl.p;
  const int heads = pl.vbatch * p.n_q_heads;
  if (2 * heads > pl.num_cus) {
    const bool most = heads <= pl.num_cus && (pl.q_len == 1 || 4 * heads > 3 * pl.num_cus);
    return most && fused_splits_fit(pl, 1) ? 1 : 0;
  }
  const int rows = p.sink + p.window + pl.k_max + pl.b0_max;  // the shortest list of the longest sequence
  const bool tight = (pl.z_half / pl.eps) * (pl.z_half / pl.eps) > 3000.0;
  if (pl.q_len == 1 && rows <= 768 && p.n_max <= (tight ? 1024 : 10240) && fused_splits_fit(pl, 1)) return 1;
  int s = 1;
  while (2 * s * heads <= pl.num_cus && s < 16) s *= 2;
  while (s >= 2 && !fused_splits_fit(pl, s)) s /= 2;
  return s >= 2 ? s : 0;
}

// Selection with the fused gather (denominator target, fresh final sample): pl.fuse_splits workgroups per head.
hipError_t launch_head_fused(const Plan& pl, const void* v, const int32_t* block_table, const int32_t* seq_lens,
                             const uint64_t* seq_seeds, void* ws, int32_t* out_idx, int32_t* out_counts,
                             double* out_budget_raw, float* out_stats, float* out_o, float* out_lse, bool pre_made,
                             hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  const vatt_params& p = pl.p;
  if (pre_made) {  // workgroups of the score launch made the first batches (prework_job)
    A.pre_tok = reinterpret_cast<uint4*>(static_cast<char*>(ws) + pl.off_pre_tok);
    A.pre_flags = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pl.off_pre_flags);
  }
  A.v = static_cast<const uint16_t*>(v);
  A.L = pl.kv_v;
  A.L.block_table = block_table;
  A.part = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_gather_part);
  A.out_o = out_o;
  A.out_lse = out_lse;
  A.splits = pl.fuse_splits;
  A.split_shift = 0;
  while ((1 << A.split_shift) < pl.fuse_splits) ++A.split_shift;
  A.group = pl.group;
  A.glist_cap = fused_glist_cap(pl, pl.fuse_splits);
  A.dlist_cap = fused_dlist_cap(pl, pl.fuse_splits);
  const HeadKernel kernel = fused_kernel_for(p.head_dim, p.kv_layout == VATT_LAYOUT_PAGED, pl.fuse_splits == 1, head_options(pl));
  hipLaunchKernelGGL(kernel, dim3(p.n_q_heads, pl.vbatch, pl.fuse_splits), dim3(kHeadThreads),
                     fused_head_lds_bytes(pl, pl.fuse_splits), st, A);
  return hipGetLastError();
}

}  // namespace vatt
