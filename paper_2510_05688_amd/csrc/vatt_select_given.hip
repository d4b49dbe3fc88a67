// Selection with a caller-supplied top-k set: the kernel of both phases, with the scores of the listed tokens
// (first phase) or the gather (second phase) fused in at small batch, and its launchers.
#include <algorithm>

#include "vatt_select.h"

namespace vatt {
namespace {

// ---------------------------------------------------------------------------
// Selection with a caller-supplied top-k set (no score row exists).
//   phase 0: I_t = the supplied tokens that lie in the middle region, without repeats; ascending list;
//            sizes of Algorithm 1 from |I_t|; base sample drawn (its weights are not known yet).
//   phase 1: with the scores of I_f and I_bs at hand (sparse list): maximum, D_f, base-sample sums, budget of
//            Algorithm 2 for the denominator target, final sample.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int base_count_of(int n_s, const SelectParams& p) {
  int b0 = p.base_abs > 0 ? p.base_abs : (int)floor(p.base_frac * (double)n_s);
  b0 = b0 < 2 ? 2 : b0;
  return b0 > n_s ? n_s : b0;
}

// Whether the final sample's first batch of draws is made before its budget is known.  Budgets grow with (z / epsilon)^2; where that is
// large (epsilon below 0.028 at delta 0.05) they mostly go beyond what a batch of this size holds or take the whole residual, unless the
// residual is so short that the batch holds half of it, and with that any sample (beyond half the complement is drawn).  There a batch
// of the right size, made when the budget is known, is better.  Measured, us per call, ahead / when known: 1 x 8K tokens at epsilon 0.02
// 31.7 / 30.7, 4 x 4K 44.0 / 42.6, 16 x 8K 98.2 / 95.8, 3 x 3K at 0.01 39.8 / 38.8, with the random cache 38.9 / 36.8, though 3 x 1.5K at
// 0.02 32.7 / 33.6; at 0.03 4 x 4K 32.5 / 33.2, 1 x 32K 27.1 / 28.1; of 0.7K at 0.02 28.5 / 29.0.
__device__ __forceinline__ bool draw_ahead(const HeadArgs& A, const HeadSizes& hs) {
  return !A.large_budgets || likely_blocks(kHeadThreads, hs, final_draws(hs)) <= kHeadThreads / 2;
}

// FD = 0: selection only.  FD = head dimension (phase 1 only): the gather is fused in for small batches, as in
// head_kernel: every head gets A.splits workgroups (blockIdx.z), each of which runs the whole second phase
// (identical results in all of them), keeps every A.splits-th token of the final sample in LDS, and gathers
// that share and a contiguous run of I_f: scores of I_f from the sparse list, scores of the sampled tokens from
// their K rows, V rows, running maximum per lane group (no head maximum bounds the sampled scores); one partial
// (N, D, maximum) per workgroup for given_merge_kernel.
// PHASE is a constant of the kernel: what both phases could share is little, and values that only one of them loads would be
// waited for where the paths meet.
template <int NT, int FD, bool PAGED, int PHASE, bool BESIDE = false>
__device__ __forceinline__ void given_topk(const HeadArgs& A) {
  using O = HeadOps<NT>;
  using HeadSmem = typename O::HeadSmem;
  using Sampler = typename O::Sampler;
  constexpr int SW = NT / kWave;
  constexpr bool kFused = FD > 0;
  extern __shared__ __align__(16) unsigned char dyn_smem[];
  __shared__ float s_wf[16];
  const uint32_t split = kFused ? blockIdx.z : 0u, shift = kFused ? (uint32_t)A.split_shift : 0u;
  const bool writer = split == 0u;
  const int h = head_of_block((int)blockIdx.x, A.Hq, A.Hkv, A.group_major), b = blockIdx.y;
  const int bh = b * A.Hq + h;
  const int tid = threadIdx.x;
  const int seq = seq_of_pair(b, A.q_len), qtok = b - seq * A.q_len;  // (sequence, query token) of a multi-query step
  const int n = max(min(max(A.seq_lens[seq], 1), A.n_max) - (A.q_len - 1 - qtok), 1);  // clamp, then the causal cut
  HeadSizes hs = head_sizes(n, A.sp);
  const int words = (n + 31) >> 5;
  HeadSmem& sm = *reinterpret_cast<HeadSmem*>(dyn_smem);
  // (the fused forms have a second scratch bitmap and mail slots for the final sample's stream, where the first phase makes both first
  // batches at once)
  const HeadLds at = head_lds<NT, kFused>(A.n_max);
  const SamplerLds apart = sampler_lds<NT>(A.n_max);
  uint32_t* lds = reinterpret_cast<uint32_t*>(dyn_smem);
  uint32_t *bm_f = lds + (kFused ? at.bm_f : apart.bm_f), *taken = lds + (kFused ? at.taken0 : apart.taken), *taken1 = lds + at.taken1;
  uint32_t *scratch = lds + (kFused ? at.scratch0 : apart.scratch), *scratch1 = lds + at.scratch1;
  uint32_t *wpre = lds + (kFused ? at.wpre : apart.wpre), *mail = lds + (kFused ? at.mail0 : apart.mail), *mail1 = lds + at.mail1;
  // fused gather (second phase): this workgroup's share of the final sample, and the cross-wave sums
  uint32_t* dlist = lds + at.lists;
  float* g_red = reinterpret_cast<float*>(dlist + (kFused ? A.dlist_cap : 0));
  // fused scores (first phase): this workgroup's run of I_f, its share of the base sample and, for a base sample
  // from the random cache, the slots of that share
  uint32_t* glist = lds + at.lists;
  uint32_t* blist = glist + (kFused ? A.glist_cap : 0);
  uint32_t* bslot = blist + (kFused ? A.dlist_cap : 0);
  int32_t* idx = A.out_idx + (int64_t)bh * A.idx_cap;
  const float* sp = A.sparse + (int64_t)bh * A.idx_cap;
  const int mid_len = hs.mid_hi - hs.mid_lo;
  const int kvh = div_group(h, A.group);

  // What can be asked for before anything is worked out comes first, and the first batch of draws, which depends on the seed,
  // the head and the length only, is made while it is under way.
  HeadRec rec = {};
  uint4 pre_t = make_uint4(0u, 0u, 0u, 0u);
  uint32_t pre_f = 0u, pre_all = 0u;
  if constexpr (PHASE != 0) {
    rec = A.head_rec[bh];
    if constexpr (kFused) {
      pre_t = A.pre_tok[(int64_t)bh * NT + tid];
      pre_f = A.pre_flags[(int64_t)bh * NT + tid];
      pre_all = A.pre_flags[(int64_t)bh * NT];  // (the same word for the whole workgroup)
    }
  }
  const int cnt = PHASE == 0 ? min(max(A.given_cnt[bh], 0), A.k_max) : rec.k;  // entries of the list of top-k tokens
  // (loads without a condition around them, of something valid where there is nothing to load: an empty list of the caller's may
  // have no memory behind it)
  const int32_t* list = PHASE != 0 ? idx + A.seg_topk : list_or(A.given_idx, (int64_t)bh * A.k_max, cnt, idx);
  // (four entries per thread are read before any is used: a read behind a condition waits for the one before)
  constexpr int U = 4;
  auto load_list = [&](int t0, int (&g)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      g[u] = list[list_entry(t0 + u * NT + tid, cnt)];
    }
  };
  int g_first[U];
  load_list(0, g_first);
  // first phase: the random cache's slots, as many per thread whatever it holds
  const unsigned char* cache_rec = PHASE == 0 && A.rcache ? cache_record(A.rcache, A.rc, seq, A.Hkv, kvh) : nullptr;
  const int32_t* ctok = cache_rec ? reinterpret_cast<const int32_t*>(cache_rec + 16) : idx;
  const int c_last = cache_rec ? A.rc.slots - 1 : 0;
  const int c_per = cache_rec ? (A.rc.slots + NT - 1) / NT : 0;
  int c_cnt = 0, c_first[U];
  auto load_slots = [&](int sb, int (&tk)[U]) {
#pragma unroll
    for (int j = 0; j < U; ++j) tk[j] = ctok[min(sb + j, c_last)];
  };
  if constexpr (PHASE == 0) {
    load_slots(tid * c_per, c_first);
    if (cache_rec) c_cnt = min(max(*reinterpret_cast<const int32_t*>(cache_rec), 0), A.rc.slots);
  }
  // second phase: scores of [sink | window | top-k | base sample], a few per thread
  // (places by arithmetic and loads without a condition around them, so that a thread's loads go out together;
  // a slot beyond the list repeats the last entry and then counts as -inf)
  const int n_fix1 = hs.n_sink + hs.n_win + rec.k, n_all = n_fix1 + (rec.n_s > 0 ? base_count_of(rec.n_s, A.sp) : 0);
  // (what is done with a loaded value stands where it is used: next to the load it would be waited for there)
  auto load_scores = [&](int base, float (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = min(base + u * NT + tid, n_all - 1);
      const uint32_t fixed = (uint32_t)fixed_place(p, hs.n_sink, hs.n_win, A.seg_sink, A.seg_win, A.seg_topk);
      v[u] = sp[p < n_fix1 ? fixed : (uint32_t)A.seg_base + (uint32_t)(p - n_fix1)];
    }
  };
  auto mask_scores = [&](int base, float (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = base + u * NT + tid < n_all ? v[u] : -INFINITY;
  };
  float v_first[U];  // the first four stay in registers
  if constexpr (PHASE != 0) load_scores(0, v_first);
  // second phase, fused gather: the rows of this workgroup's run of I_f (LPR adjacent lanes hold one row, NG rows per round, UF
  // rounds in flight; places, tokens, block-table entries and rows each in a loop of their own over the UF slots: no branch
  // per row; a slot beyond the list repeats its last entry and adds nothing).  Their tokens and scores are asked for here, the
  // rows after the draws, and they are added at the end.
  constexpr int LPR = kFused ? FD / 8 : 16;
  constexpr int NG = NT / LPR;
  constexpr int UF = 8;
  const int g_sub = tid % LPR, g_grp = tid / LPR;
  const int run1 = (n_fix1 + (int)A.splits - 1) >> shift;
  const int f_lo = min((int)split * run1, n_fix1), f_hi = min(f_lo + run1, n_fix1);
  int f_tok[UF];
  float f_sc[UF];
  uint4 f_v[UF];
  auto load_fixed = [&](int j0) {
#pragma unroll
    for (int u = 0; u < UF; ++u) {
      const uint32_t place = (uint32_t)fixed_place(max(min(j0 + g_grp + u * NG, f_hi - 1), 0), hs.n_sink, hs.n_win, A.seg_sink, A.seg_win, A.seg_topk);
      f_tok[u] = idx[place];
      f_sc[u] = sp[place];
    }
  };
  // f(from, to) for the quarters of the UF rounds that a batch of `rows` rows (a whole-workgroup value) has
  auto each_part = [](int rows, auto&& f) {
    f(Int<0>{}, Int<UF / 4>{});
    if (rows > UF / 4 * NG) f(Int<UF / 4>{}, Int<UF / 2>{});
    if (rows > UF / 2 * NG) f(Int<UF / 2>{}, Int<UF>{});
  };
  auto load_fixed_rows = [&](int j0) {
    int blk[UF];
#pragma unroll
    for (int u = 0; u < UF; ++u) {
      f_tok[u] = min(max(f_tok[u], 0), n - 1);
      blk[u] = kv_block<PAGED>(A.L, seq, f_tok[u]);
    }
    each_part(f_hi - j0, [&](auto from, auto to) {
#pragma unroll
      for (int u = decltype(from)::value; u < decltype(to)::value; ++u)
        f_v[u] = load_stream_16(A.v + kv_row_offset_in<PAGED>(A.L, seq, kvh, f_tok[u], blk[u]) + g_sub * 8);
    });
  };
  if constexpr (kFused && PHASE != 0) load_fixed(f_lo);

  for (int w = tid; w < words; w += NT) {
    bm_f[w] = 0;
    taken[w] = 0;
    scratch[w] = 0;
    if constexpr (kFused && PHASE == 0) {
      taken1[w] = 0;
      scratch1[w] = 0;
    }
  }
  __syncthreads();
  Sampler S;
  S.taken = taken;
  S.scratch = scratch;
  S.mail = mail;
  S.bm_f = bm_f;
  S.wpre = wpre;
  S.row = nullptr;
  S.seed = A.seq_seeds[seq];
  S.stream = PHASE == 0 ? 0u : 1u;
  S.head = (uint32_t)h;
  S.query = (uint32_t)qtok;
  S.L = (uint32_t)max(mid_len, 1);
  S.thr = (0u - S.L) % S.L;  // 2^32 mod L
  {
    const uint64_t dflt = 64ull * (uint64_t)S.L + 4096ull;
    S.cap = (uint32_t)min(A.draw_cap ? (uint64_t)A.draw_cap : dflt, 0x80000000ull);
  }
  S.m = 0.f;
  S.dbg = nullptr;
  DrawBatch spec = {};
  bool have_spec = false, pair_made = false;
  int blocks1 = 0;
  // leaves a Philox block's four draws of the final sample's first batch for the second phase
  auto store_final = [&](int block, const DrawBatch& B, bool made) {
    const int64_t place = (int64_t)bh * NT + block;
    A.pre_tok[place] = make_uint4(B.tok[0], B.tok[1], B.tok[2], B.tok[3]);
    A.pre_flags[place] = pre_pack(B, made);
  };
  // Philox blocks of the final sample's first batch: enough for the base sample's size, and for a larger sample as many as half
  // of the threads make
  auto final_blocks = [&](const HeadSizes& he) {
    return max(likely_blocks(A.small_batches ? kSmallBatchBlocks : NT, he, base_draws(he)),
               ahead_blocks<NT>(A.small_batches, he, final_draws(he)));
  };
  if constexpr (kFused && PHASE != 0) {
    // made by a workgroup of the first phase, under its loads of K rows
    have_spec = pre_made_of(pre_all);
    spec.blocks = pre_blocks(pre_all);
    spec.ok = pre_ok(pre_f);
    spec.first = pre_first(pre_f);
    const uint32_t tk[4] = {pre_t.x, pre_t.y, pre_t.z, pre_t.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      spec.tok[e] = min(max(tk[e], (uint32_t)hs.mid_lo), (uint32_t)max(hs.mid_hi - 1, hs.mid_lo));
      if (have_spec && ((spec.ok >> e) & 1u)) O::mark_bit(taken, spec.tok[e]);
    }
  } else {
    // (first phase: the list's length stands for the size of the set; the batch's size changes no result)
    HeadSizes he = hs;
    he.k = min(cnt, max(mid_len, 0));
    he.n_s = mid_len - he.k;
    he.b0 = he.n_s > 0 ? base_count_of(he.n_s, A.sp) : 0;
    have_spec = he.n_s > 0 && he.b0 < he.n_s && (PHASE == 0 ? !A.rcache : !A.nested && draw_ahead(A, he));
    const int blocks = PHASE == 0 ? likely_blocks(A.small_batches ? kSmallBatchBlocks : NT, he, base_draws(he)) : final_blocks(he);
    if constexpr (kFused && PHASE == 0) {
      // first batches of both samples at once where half of the workgroup holds each (as in the kernel of the scored path):
      // small steps, whose rows would not cover the second one (below), 28.1 -> 27.4 us for 3 x 0.7K tokens
      blocks1 = final_blocks(he);
      pair_made = have_spec && blocks <= NT / 2 && blocks1 <= NT / 2 && draw_ahead(A, he);
      if (pair_made) {
        Sampler S1 = S;
        S1.taken = taken1;
        S1.scratch = scratch1;
        S1.mail = mail1;
        S1.stream = 1u;
        const bool upper = tid >= NT / 2;
        DrawBatch mine = {};
        O::make_batch(mine, upper ? S1 : S, hs, 0u, upper ? blocks1 : blocks, false, false, sm, upper ? tid - NT / 2 : tid);
        spec = mine;
        spec.blocks = blocks;
        spec.ok = upper ? 0u : mine.ok;
        spec.first = upper ? 0u : mine.first;
        if ((int)split == A.splits - 1) {
          mine.blocks = blocks1;
          mine.ok = upper ? mine.ok : 0u;
          mine.first = upper ? mine.first : 0u;
          store_final(upper ? tid - NT / 2 : tid + NT / 2, mine, true);
        }
      }
    }
    if (have_spec && !pair_made) O::make_batch(spec, S, hs, 0u, blocks, false, false, sm, tid);
  }
  if constexpr (kFused && PHASE != 0) load_fixed_rows(f_lo);
  auto mark = [&](int t0, const int (&g)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t0 + u * NT + tid < cnt && g[u] >= hs.mid_lo && g[u] < hs.mid_hi) O::mark_bit(bm_f, (uint32_t)g[u]);
  };
  mark(0, g_first);
  for (int t0 = U * NT; t0 < cnt; t0 += U * NT) {
    int g[U];
    load_list(t0, g);
    mark(t0, g);
  }
  __syncthreads();
  const int k_eff = PHASE == 0 ? (int)O::word_prefix(bm_f, words, wpre, sm, &sm.scan_once[0]) : rec.k;
  hs.k = k_eff;
  hs.n_s = mid_len - k_eff;
  hs.b0 = hs.n_s > 0 ? base_count_of(hs.n_s, A.sp) : 0;

  // (first phase fused with the scores: the run of [sink | window | top-k) this workgroup scores)
  int f0_lo = 0, f0_hi = 0;
  if (kFused && PHASE == 0) {
    const int n_f = hs.n_sink + hs.n_win + k_eff;
    const int run = min((n_f + (int)A.splits - 1) >> shift, A.glist_cap);
    f0_lo = min((int)split * run, n_f);
    f0_hi = min(f0_lo + run, n_f);
  }

  if constexpr (PHASE == 0) {
    // every entry finds its own place: the members below it, from the word prefix and the bits below its own (a repeated token
    // writes the same place twice)
    auto place = [&](int t0, const int (&g)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (t0 + u * NT + tid < cnt && g[u] >= hs.mid_lo && g[u] < hs.mid_hi) {
          const uint32_t pos = wpre[g[u] >> 5] + (uint32_t)__popc(bm_f[g[u] >> 5] & ((1u << (g[u] & 31)) - 1u));
          if (writer && pos < (uint32_t)A.k_max) idx[A.seg_topk + pos] = g[u];
          if (kFused) {
            const int p = hs.n_sink + hs.n_win + (int)pos;  // place in [sink | window | top-k)
            if (p >= f0_lo && p < f0_hi) glist[p - f0_lo] = (uint32_t)g[u];
          }
        }
      }
    };
    place(0, g_first);
    for (int t0 = U * NT; t0 < cnt; t0 += U * NT) {
      int g[U];
      load_list(t0, g);
      place(t0, g);
    }
    for (int i = tid; i < hs.n_sink; i += NT) {
      if (writer) idx[A.seg_sink + i] = i;
      if (kFused && i >= f0_lo && i < f0_hi) glist[i - f0_lo] = (uint32_t)i;
    }
    for (int i = tid; i < hs.n_win; i += NT) {
      if (writer) idx[A.seg_win + i] = hs.mid_hi + i;
      const int p = hs.n_sink + i;
      if (kFused && p >= f0_lo && p < f0_hi) glist[p - f0_lo] = (uint32_t)(hs.mid_hi + i);
    }
    int flags = 0;
    bool cached = false;
    if (hs.n_s > 0 && cache_rec) {
      // base sample = the first b0 cached tokens, in slot order, that are residual tokens of this head; the
      // cache is used only when it holds that many
      const int s0 = min(tid * c_per, c_cnt), s1 = min(s0 + c_per, c_cnt);
      // a thread's slots four at a time: their tokens are read together, then their bitmap words together
      // (bit j of the result: slot sb + j holds a residual token; the token comes back in tk[j])
      auto residual4 = [&](int sb, int (&tk)[U]) -> uint32_t {
        uint32_t w[U], r4 = 0;
        if (sb == s0) {
#pragma unroll
          for (int j = 0; j < U; ++j) tk[j] = c_first[j];
        } else {
          load_slots(sb, tk);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) w[j] = bm_f[min(max(tk[j], 0), n - 1) >> 5];  // (a token outside the sequence fails the range test below)
#pragma unroll
        for (int j = 0; j < U; ++j)
          r4 |= ((sb + j < s1 && tk[j] >= hs.mid_lo && tk[j] < hs.mid_hi && !((w[j] >> (tk[j] & 31)) & 1u)) ? 1u : 0u) << j;
        return r4;
      };
      uint32_t mine = 0;
      for (int sb = s0; sb < s1; sb += U) {
        int tk[U];
        mine += (uint32_t)__popc(residual4(sb, tk));
      }
      uint32_t total;
      uint32_t pos = block_exclusive_scan_once<NT>(mine, &total, sm.scan_once[1]);
      cached = total >= (uint32_t)hs.b0;
      if (cached) {
        int32_t* slot_of = A.base_slot + (int64_t)bh * A.b0_max;
        const uint32_t lim = (uint32_t)min(hs.b0, A.b0_max);
        for (int sb = s0; sb < s1 && pos < lim; sb += U) {
          int tk[U];
          const uint32_t r4 = residual4(sb, tk);
#pragma unroll
          for (int j = 0; j < U; ++j) {
            if (((r4 >> j) & 1u) && pos < lim) {
              if (writer) {
                idx[A.seg_base + pos] = tk[j];
                slot_of[pos] = sb + j;
              }
              if (kFused && (pos & ((1u << shift) - 1u)) == split && (pos >> shift) < (uint32_t)A.dlist_cap) {
                blist[pos >> shift] = (uint32_t)tk[j];
                bslot[pos >> shift] = (uint32_t)(sb + j);
              }
              ++pos;
            }
          }
        }
        flags |= kFlagBaseFromCache;
      }
    }
    if (hs.n_s > 0 && !cached) {
      __syncthreads();  // (the sampler may take the word prefixes' place)
      Emit E0 = emit_to(idx + A.seg_base, (uint32_t)A.b0_max);
      if (kFused) {
        E0.global = writer;
        E0.lds = blist;
        E0.lds_cap = (uint32_t)A.dlist_cap;
        E0.shift = shift;
        E0.split = split;
      }
      const int f = O::draw_sample(S, hs, (uint32_t)hs.b0, spec, have_spec, A.small_batches, E0, nullptr, nullptr, sm, 0u, 0u, true);
      flags |= ((f & 1) ? kFlagBaseComplement : 0) | ((f & 2) ? kFlagBaseBatches : 0) | ((f & 4) ? kFlagDrawCap : 0);
      if (!kFused && A.ascending && !(f & 1))
        O::sort_ascending(idx + A.seg_base, (uint32_t)min(hs.b0, A.b0_max), scratch, wpre, n, sm);
    }
    if (tid == 0 && writer) {
      HeadRec r;
      r.m = 0.f;
      r.scale = 0.f;
      r.n = n;
      r.n_sink = hs.n_sink;
      r.n_win = hs.n_win;
      r.k = k_eff;
      r.b = hs.b0;  // the score pass walks the base sample
      r.n_s = hs.n_s;
      r.b_keep = 0;
      r.base_cached = cached ? 1 : 0;
      r.tail_by_token = 0;
      A.head_rec[bh] = r;
      A.out_counts[(int64_t)bh * 8 + 7] = flags;
    }
    if constexpr (kFused) {
      // ---- the scores of this workgroup's share of I_f and of the base sample (denominator target) ----
      // s_i = sm_scale <K[i], q>, written to the tokens' places of the sparse list; rows as in the gather below:
      // tokens, block-table entries and rows each in a loop of their own over the slots in flight
      __syncthreads();  // the lists of this workgroup's share are complete
      float* spw = const_cast<float*>(A.sparse) + (int64_t)bh * A.idx_cap;
      uint32_t qw[4];
      {
        const uint4 t = *reinterpret_cast<const uint4*>(A.gq + (int64_t)bh * FD + g_sub * 8);
        qw[0] = t.x;
        qw[1] = t.y;
        qw[2] = t.z;
        qw[3] = t.w;
      }
      auto score_of = [&](const uint4& kv) -> float {
        float a = 0.f;
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv.x), __builtin_bit_cast(bf16x2_t, qw[0]), a, false);
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv.y), __builtin_bit_cast(bf16x2_t, qw[1]), a, false);
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv.z), __builtin_bit_cast(bf16x2_t, qw[2]), a, false);
        a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv.w), __builtin_bit_cast(bf16x2_t, qw[3]), a, false);
        return group_sum<LPR>(a) * A.sm_scale + 0.0f;
      };
      const int my_nf = f0_hi - f0_lo;
      int my_nb = hs.n_s > 0 && hs.b0 > (int)split ? (int)(((uint32_t)hs.b0 - split + ((1u << shift) - 1u)) >> shift) : 0;
      my_nb = min(my_nb, A.dlist_cap);
      auto load_listed = [&](const uint32_t* list, int j0, int count, uint4 (&kv)[UF]) {
        int tok[UF], blk[UF];
#pragma unroll
        for (int u = 0; u < UF; ++u) tok[u] = (int)min(list[min(j0 + u * NG, count - 1)], (uint32_t)(n - 1));
#pragma unroll
        for (int u = 0; u < UF; ++u) blk[u] = kv_block<PAGED>(A.Lk, seq, tok[u]);
#pragma unroll
        for (int u = 0; u < UF; ++u)
          kv[u] = load_stream_16(A.gk + kv_row_offset_in<PAGED>(A.Lk, seq, kvh, tok[u], blk[u]) + g_sub * 8);
      };
      auto load_base = [&](int j0, uint4 (&kv)[UF]) {
        if (cached) {
          // the copies of the rows in the cache: rows of neighbouring slots, shared by the group's heads
          int slot[UF];
#pragma unroll
          for (int u = 0; u < UF; ++u) slot[u] = (int)min(bslot[min(j0 + u * NG, my_nb - 1)], (uint32_t)(A.rc.slots - 1));
#pragma unroll
          for (int u = 0; u < UF; ++u)
            kv[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(cache_rec + A.rc.off_k) +
                                                    (int64_t)slot[u] * FD + g_sub * 8);
        } else {
          load_listed(blist, j0, my_nb, kv);
        }
      };
      // (the first rows of both lists are under way together; a lane group beyond a list's end stays out, and with it whole waves:
      // small base samples fill one or two of eight, 3 x 0.7K tokens 24.3 -> 23.8 us per call, 1 x 4K of 64 columns 23.9 -> 22.8)
      uint4 kf[UF], kb[UF];
      if (g_grp < my_nf) load_listed(glist, g_grp, my_nf, kf);
      if (g_grp < my_nb) load_base(g_grp, kb);
      if ((int)split == A.splits - 1 && !pair_made) {
        // The first batch of the final sample's draws, for all workgroups of the head in the second phase, where it would
        // stand in front of everything else.  Here it is made while the rows are on their way.
        const bool make = hs.n_s > 0 && hs.b0 < hs.n_s && draw_ahead(A, hs);
        DrawBatch mine = {};
        if (make) {
          for (int w = tid; w < words; w += NT) taken[w] = 0;  // (the base sample's)
          __syncthreads();
          Sampler S1 = S;
          S1.stream = 1u;
          O::make_batch(mine, S1, hs, 0u, final_blocks(hs), false, false, sm, tid);
        }
        store_final(tid, mine, make);
      }
      for (int j0 = g_grp; j0 < my_nf; j0 += NG * UF) {
        if (j0 != g_grp) load_listed(glist, j0, my_nf, kf);
#pragma unroll
        for (int u = 0; u < UF; ++u) {
          const float sc = score_of(kf[u]);
          const int j = j0 + u * NG;
          if (j < my_nf && g_sub == 0)
            spw[fixed_place(f0_lo + j, hs.n_sink, hs.n_win, A.seg_sink, A.seg_win, A.seg_topk)] = sc;
        }
      }
      for (int j0 = g_grp; j0 < my_nb; j0 += NG * UF) {
        if (j0 != g_grp) load_base(j0, kb);
#pragma unroll
        for (int u = 0; u < UF; ++u) {
          const float sc = score_of(kb[u]);
          const int j = j0 + u * NG;
          if (j < my_nb && g_sub == 0) spw[A.seg_base + (((int64_t)j << shift) | split)] = sc;
        }
      }
    }
  } else {
  // ---- phase 1 ----
  const int n_fix = n_fix1;
  float v_max = -INFINITY;
  mask_scores(0, v_first);
#pragma unroll
  for (int u = 0; u < U; ++u) v_max = fmaxf(v_max, v_first[u]);
  for (int base = NT * U; base < n_all; base += NT * U) {
    float v[U];
    load_scores(base, v);
    mask_scores(base, v);
#pragma unroll
    for (int u = 0; u < U; ++u) v_max = fmaxf(v_max, v[u]);
  }
  v_max = wave_max(v_max);
  if ((tid & 63) == 0) s_wf[tid >> 6] = v_max;
  // The accepted ones of the first batch of draws are counted by one scan, whose barrier serves the maximum too.  (Their rows are
  // asked for when the budget is known.  With those of the first b0, which it cannot drop unless the sample is a complement, requested
  // before it as in the kernel of the scored path, the kernel takes 190 registers instead of 124 and a seventh more code, and every size is
  // slower: 1 x 32K tokens 26.3 us per call instead of 26.1, 1 x 8K 23.8 instead of 22.7, 3 x 0.7K 25.7 instead of 24.3.)
  const uint32_t smask = (1u << shift) - 1u;
  auto share_of = [&](uint32_t c) { return c > split ? (int)((c - split + smask) >> shift) : 0; };
  const bool usual = have_spec && 2 * hs.b0 <= hs.n_s && (kFused || !A.ascending);
  const uint32_t acc_bits = usual ? spec.first & ~O::test_bits4(bm_f, spec.tok) : 0u;
  uint32_t tot1;
  const uint32_t acc_pos = block_exclusive_scan_once<NT>((uint32_t)__popc(acc_bits), &tot1, sm.scan_once[2]);
  float m = s_wf[0];
#pragma unroll
  for (int w = 1; w < SW; ++w) m = fmaxf(m, s_wf[w]);
  double acc_f = 0.0, acc_w = 0.0, acc_w2 = 0.0;
  for (int base = 0; base < n_all; base += NT * U) {
    float v[U];
    if (base == 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = v_first[u];
    } else {
      load_scores(base, v);  // (a second read of a few values, only for lists beyond 2048 entries)
      mask_scores(base, v);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = base + u * NT + tid;
      const double w = (double)__expf(v[u] - m);  // 0 for the slots beyond the list
      acc_f += p < n_fix ? w : 0.0;
      acc_w += p < n_fix ? 0.0 : w;
      acc_w2 += p < n_fix ? 0.0 : w * w;
    }
  }
  double sums[3] = {acc_f, acc_w, acc_w2};
  O::block_sum_post(sums, sm);
  __syncthreads();
  O::block_sum_get(sums, sm);
  const double D_f = sums[0];
  double sigma2 = 0.0, b_star = 0.0, D_hat = D_f, tr_sigma = 0.0, nhat_sq = 0.0;
  int bfin = 0;
  if (hs.n_s > 0) {
    const double b0d = (double)hs.b0, ns = (double)hs.n_s;
    double rho_N = 0.0;
    if (A.target != VATT_TARGET_D) {
      // numerator statistics left by the score kernel of the listed tokens, one partial per split, each in
      // units of its own maximum: brought to the head's maximum m (the largest of them) and added
      const int d = A.head_dim;
      const int stride = 2 * d + 4;
      const float* vp = A.given_vstat + (int64_t)bh * A.given_splits * stride;
      double t3[3] = {0.0, 0.0, 0.0};
      if (tid < d) {
        double nf = 0.0, r1 = 0.0;
        for (int s2 = 0; s2 < A.given_splits; ++s2) {
          const float ms = vp[s2 * stride + 2 * d + 1];
          const double f = ms > -INFINITY ? exp((double)ms - (double)m) : 0.0;
          nf += (double)vp[s2 * stride + tid] * f;
          r1 += (double)vp[s2 * stride + d + tid] * f;
        }
        const double nh = nf + ns * r1 / b0d;
        t3[0] = nh * nh;
        t3[1] = r1 * r1;
      }
      if (tid == 0) {
        for (int s2 = 0; s2 < A.given_splits; ++s2) {
          const float ms = vp[s2 * stride + 2 * d + 1];
          const double f = ms > -INFINITY ? exp((double)ms - (double)m) : 0.0;
          t3[2] += (double)vp[s2 * stride + 2 * d] * f * f;
        }
      }
      O::block_sum(t3, sm);
      nhat_sq = t3[0];
      rho_N = numerator_rho(hs.n_s, hs.b0, t3[1], t3[2], nhat_sq, &tr_sigma);
    }
    const Budget bud = algorithm2_budget(A, hs.n_s, hs.b0, D_f, sums[1], sums[2], rho_N, 0.0);
    sigma2 = bud.sigma2;
    b_star = bud.b_star;
    bfin = bud.b;
    D_hat = bud.D_hat;
  }
  int flags = 0;
  const bool fast_dyn = usual && (uint32_t)bfin <= tot1 && 2 * bfin <= hs.n_s;  // the first batch of draws holds the sample
  if (fast_dyn) {
    uint32_t pos = acc_pos;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool a = (acc_bits >> e) & 1u;
      if (a && pos < (uint32_t)bfin) {
        if (writer && pos < (uint32_t)A.b_max) idx[A.seg_dyn + pos] = (int32_t)spec.tok[e];
        if (kFused && (pos & smask) == split && (pos >> shift) < (uint32_t)A.dlist_cap) dlist[pos >> shift] = spec.tok[e];
      }
      pos += a ? 1u : 0u;
    }
    // (a first batch of the sample's own size would not have held it: a thread makes a block, so whole waves count)
    uint32_t held = 0;
    for (int w = 0; w < O::first_blocks(A.small_batches, (uint32_t)bfin) / kWave; ++w) held += sm.scan_once[2].wave_total[w];
    if (held < (uint32_t)bfin) flags |= kFlagDynBatches;
  }
  if (bfin > 0 && !fast_dyn) {
    Emit E1 = emit_to(idx + A.seg_dyn, (uint32_t)A.b_max);
    if (kFused) {
      E1.global = writer;
      E1.lds = dlist;
      E1.lds_cap = (uint32_t)A.dlist_cap;
      E1.shift = shift;
      E1.split = split;
    }
    const int f = (!kFused && A.nested)
                      ? O::draw_nested(S, hs, (uint32_t)hs.b0, (uint32_t)bfin, bm_f, idx + A.seg_base,
                                       idx + A.seg_dyn, (uint32_t)A.b_max, A.small_batches, sm)
                      : O::draw_sample(S, hs, (uint32_t)bfin, spec, have_spec, A.small_batches, E1, nullptr, nullptr, sm, 0u, 0u, true);
    flags |= ((f & 1) ? kFlagDynComplement : 0) | ((f & 2) ? kFlagDynBatches : 0) | ((f & 4) ? kFlagDrawCap : 0);
    if (!kFused && A.ascending && !A.nested && !(f & 1))
      O::sort_ascending(idx + A.seg_dyn, (uint32_t)min(bfin, A.b_max), scratch, wpre, n, sm);
  }
  if (tid == 0 && writer) {
    int32_t* c = A.out_counts + (int64_t)bh * 8;
    c[0] = hs.n_sink;
    c[1] = hs.n_win;
    c[2] = k_eff;
    c[3] = hs.b0;
    c[4] = bfin;
    c[5] = hs.n_s;
    c[6] = n;
    c[7] = c[7] | flags;
    if (A.out_budget_raw) A.out_budget_raw[bh] = b_star;
    if (A.out_stats) {
      float* st = A.out_stats + (int64_t)bh * 4;
      st[0] = (float)D_hat;
      st[1] = (float)sigma2;
      st[2] = (float)tr_sigma;
      st[3] = (float)nhat_sq;
      // (in units of exp(-m) with m the largest score among I_f and I_bs, which is HeadRec.m and out_lse's shift)
    }
    HeadRec r;
    r.m = m;
    r.scale = bfin > 0 ? (float)((double)hs.n_s / (double)bfin) : 0.f;
    r.n = n;
    r.n_sink = hs.n_sink;
    r.n_win = hs.n_win;
    r.k = k_eff;
    r.b = bfin;
    r.n_s = hs.n_s;
    r.b_keep = (A.nested && bfin > 0) ? hs.b0 : 0;
    r.base_cached = 0;
    r.tail_by_token = 0;
    // (with the gather fused in nothing reads the record again, and the head's other workgroups may still be
    // reading the first phase's)
    HeadRec* to = A.head_rec + bh;
    if (BESIDE) {  // (the other fields stay the first phase's: gather_fixed is reading them; written whole it is 0.2 us faster where nobody is)
      to->m = r.m;
      to->scale = r.scale;
      to->b = r.b;
      to->b_keep = r.b_keep;
    } else if (!kFused) {
      *to = r;
    }
  }

  if constexpr (kFused) {
    // ---- the gather of this workgroup's share ----
    __syncthreads();  // the final sample's share is complete in dlist
    uint32_t qw[4];
    {
      const uint4 t = *reinterpret_cast<const uint4*>(A.gq + (int64_t)bh * FD + g_sub * 8);
      qw[0] = t.x;
      qw[1] = t.y;
      qw[2] = t.z;
      qw[3] = t.w;
    }
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float dsum = 0.f, m_run = -INFINITY;
    auto add_row = [&](float e, const uint4& vv) {
      if (e > m_run) {
        const float f = __expf(m_run - e);  // 0 when m_run is -inf
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] *= f;
        dsum *= f;
        m_run = e;
      }
      const float wt = __expf(e - m_run);
      add_weighted_row(acc, wt, vv);
      dsum += wt;
    };
    // I_f: a contiguous run of [sink | window | top-k) per workgroup (the top-k part is in ascending token order)
    for (int j0 = f_lo; j0 < f_hi; j0 += NG * UF) {
      if (j0 != f_lo) {
        load_fixed(j0);
        load_fixed_rows(j0);
      }
      each_part(f_hi - j0, [&](auto from, auto to) {
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(to)::value; ++u)
          if (j0 + g_grp + u * NG < f_hi) add_row(f_sc[u], f_v[u]);
      });
    }
    // the final sample: every A.splits-th token, scores from the K rows, weights carry n_s / b
    const int my_nd = min(share_of((uint32_t)bfin), A.dlist_cap);
    const float tail_bias = bfin > 0 ? __logf((float)((double)hs.n_s / (double)bfin)) : 0.f;
    // (place j is always read by lane group j % NG, and a group adds its rows in rising order)
    for (int first = 0; first < my_nd; first += UF * NG) {
      const int j0 = first + g_grp;
      int tok[UF], blk[UF];
      uint4 kv[UF], vv[UF];
#pragma unroll
      for (int u = 0; u < UF; ++u) tok[u] = (int)min(dlist[min(j0 + u * NG, my_nd - 1)], (uint32_t)(n - 1));
#pragma unroll
      for (int u = 0; u < UF; ++u) blk[u] = kv_block<PAGED>(A.L, seq, tok[u]);  // (K and V share the block table)
      each_part(my_nd - first, [&](auto from, auto to) {
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(to)::value; ++u) {
          kv[u] = load_stream_16(A.gk + kv_row_offset_in<PAGED>(A.Lk, seq, kvh, tok[u], blk[u]) + g_sub * 8);
          vv[u] = load_stream_16(A.v + kv_row_offset_in<PAGED>(A.L, seq, kvh, tok[u], blk[u]) + g_sub * 8);
        }
      });
      each_part(my_nd - first, [&](auto from, auto to) {
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(to)::value; ++u) {
          // (the lanes of a group stay together: every lane of the group computes the row's score)
          float a = 0.f;
          a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv[u].x), __builtin_bit_cast(bf16x2_t, qw[0]), a, false);
          a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv[u].y), __builtin_bit_cast(bf16x2_t, qw[1]), a, false);
          a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv[u].z), __builtin_bit_cast(bf16x2_t, qw[2]), a, false);
          a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, kv[u].w), __builtin_bit_cast(bf16x2_t, qw[3]), a, false);
          const float s_row = group_sum<LPR>(a) * A.sm_scale + 0.0f;
          if (j0 + u * NG < my_nd) add_row(s_row + tail_bias, vv[u]);
        }
      });
    }
    // the lane groups of a wave to their common maximum and added, then the waves through LDS
    float M = m_run;
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) M = fmaxf(M, __shfl_xor(M, o));
    {
      const float f = m_run > -INFINITY ? __expf(m_run - M) : 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] *= f;
      dsum *= f;
    }
    add_lane_groups<LPR>(acc);
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) dsum += __shfl_xor(dsum, o);
    const int lane = tid & 63, wave = tid >> 6;
    float* g_d = g_red + SW * FD;
    float* g_m = g_d + SW;
    if (LPR == 16 || (lane & 8) == 0) {
#pragma unroll
      for (int c = 0; c < 2; ++c) g_red[wave * FD + lane_groups_column<LPR>(lane) + c] = acc[c];
    }
    if (lane == 0) {
      g_d[wave] = dsum;
      g_m[wave] = M;
    }
    __syncthreads();
    float Mall = -INFINITY;
#pragma unroll
    for (int w2 = 0; w2 < SW; ++w2) Mall = fmaxf(Mall, g_m[w2]);
    float* part = A.part + ((int64_t)bh * A.splits + split) * (FD + 4);
    if (tid < FD) {
      float a = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < SW; ++w2) a += g_red[w2 * FD + tid] * (g_m[w2] > -INFINITY ? __expf(g_m[w2] - Mall) : 0.f);
      part[tid] = a;
    }
    if (tid == 0) {
      float dt = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < SW; ++w2) dt += g_d[w2] * (g_m[w2] > -INFINITY ? __expf(g_m[w2] - Mall) : 0.f);
      part[FD] = dt;
      part[FD + 1] = Mall;
    }
  }
  }
}

template <int NT, int FD, bool PAGED, int PHASE>
__global__ __launch_bounds__(NT) void given_topk_kernel(HeadArgs A) {
  given_topk<NT, FD, PAGED, PHASE>(A);
}

// Partial sums (N, D, maximum) over a share of [sink | window | top-k): scores from the sparse list, V rows, in the manner of
// given_gather_kernel and with its running maximum, which needs nothing of the second phase.
template <int D, bool PAGED>
__device__ __forceinline__ void gather_fixed(const HeadArgs& A, int split) {
  constexpr int LPR = D / 8, RPW = kWave / LPR, WAVES = kHeadThreads / kWave, RPB = RPW * WAVES, U = 8, ROWS_W = RPW * U;
  const int h = head_of_block((int)blockIdx.x, A.Hq, A.Hkv, A.group_major), b = blockIdx.y;
  const int bh = b * A.Hq + h, kvh = div_group(h, A.group), seq = seq_of_pair(b, A.q_len);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, rsub = lane / LPR;
  const HeadRec& r = A.head_rec[bh];  // (the second phase is writing m, scale, b and b_keep)
  const int n_fix = r.n_sink + r.n_win + r.k;
  const int splits = used_splits(A.splits, n_fix, fixed_step_rows(D));
  if (split >= splits) return;
  const bool shared_rows = rows_are_shared(n_fix + (r.n_s > 0 ? base_count_of(r.n_s, A.sp) : 0), A.group_major ? A.q_len * A.group : A.q_len, r.n, A.group_major && A.group > 1 ? 3 : 2);
  const int per = (n_fix + splits - 1) / splits;
  const int p_lo = split * per, p_hi = min(p_lo + per, n_fix);
  const int32_t* idx = A.out_idx + (int64_t)bh * A.idx_cap;
  const float* sp = A.sparse + (int64_t)bh * A.idx_cap;
  const uint16_t* v_head = PAGED ? A.v : A.v + (int64_t)seq * A.L.seq_stride + (int64_t)kvh * A.L.head_stride;
  const int mine = (lane / RPW) * RPB + wave * RPW + lane % RPW;  // the row of a step that this lane prepares
  int entry_next = 0;
  float sc_next = 0.f;
  auto request = [&](int p0) {  // (beyond the range: its last place once more)
    const uint32_t place = (uint32_t)fixed_place(min(p0 + mine, p_hi - 1), r.n_sink, r.n_win, A.seg_sink, A.seg_win, A.seg_topk);
    entry_next = idx[place];
    sc_next = sp[place];
  };
  if (p_lo < p_hi) request(p_lo);
  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  float dsum = 0.f, m_run = -INFINITY;
  auto walk = [&](auto load) {
    for (int p0 = p_lo; p0 < p_hi; p0 += RPB * U) {
      const bool valid = lane < ROWS_W && p0 + mine < p_hi;
      const int tok_mine = min(max(entry_next, 0), r.n - 1);
      const float e = valid ? sc_next : -INFINITY;
      request(p0 + RPB * U);
      int tok[U], blk[U];
      uint4 vv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) tok[u] = __shfl(tok_mine, u * RPW + rsub);
#pragma unroll
      for (int u = 0; u < U; ++u) blk[u] = kv_block<PAGED>(A.L, seq, tok[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
        vv[u] = load(PAGED ? A.v + kv_row_offset_in<true>(A.L, seq, kvh, tok[u], blk[u]) + sub * 8 : v_head + ((uint32_t)tok[u] * (uint32_t)D + (uint32_t)(sub * 8)));
      __builtin_amdgcn_sched_barrier(0);
      const float m_new = fmaxf(m_run, wave_max(e));
      const float f = m_run > -INFINITY ? __expf(m_run - m_new) : 0.f;
      const float wt_mine = e == -INFINITY ? 0.f : __expf(e - m_new);  // (NaN for a NaN score: the row is not left out)
      m_run = m_new;
      dsum = dsum * f + wt_mine;
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] *= f;
      if (p0 + RPB * U > p_hi) {
        // (a row beyond the range repeats the last one, with weight 0; an Inf in it would make a NaN)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p0 + u * RPB + wave * RPW + rsub >= p_hi) vv[u] = make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add_weighted_row(acc, __shfl(wt_mine, u * RPW + rsub), vv[u]);
    }
  };
  if (shared_rows) walk(LoadShared{});
  else walk(LoadOnce{});

  // the lane groups of a wave, then the waves, each with its maximum
  add_lane_groups<LPR>(acc);
  dsum = wave_sum_f32(dsum);
  __shared__ __align__(16) float s_acc[WAVES][D];
  __shared__ float s_d[WAVES], s_m[WAVES];
  if (LPR == 16 || (lane & 8) == 0) {
#pragma unroll
    for (int c = 0; c < 2; ++c) s_acc[wave][lane_groups_column<LPR>(lane) + c] = acc[c];
  }
  if (lane == 0) {
    s_d[wave] = dsum;
    s_m[wave] = m_run;
  }
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int j = 0; j < WAVES; ++j) M = fmaxf(M, s_m[j]);
  float* part = A.part + ((int64_t)bh * A.part_slots + split) * (D + 4);
  float a = 0.f, d = 0.f;
#pragma unroll
  for (int j = 0; j < WAVES; ++j) {
    const float f = s_m[j] > -INFINITY ? __expf(s_m[j] - M) : 0.f;
    if (tid < D) a += s_acc[j][tid] * f;
    d += s_d[j] * f;
  }
  if (tid < D) part[tid] = a;
  if (tid == 0) {
    part[D] = d;
    part[D + 1] = M;
  }
}

// The second phase of a step whose gather is apart, and beside it (given_fixed_splits) in the same launch and behind the workgroups of
// the phase, the first of the third grid dimension, the gather of I_f, which waits for nothing that the phase finds out: a phase
// is a chain of 9 us that leaves memory idle.
template <int D, bool PAGED>
__global__ __launch_bounds__(kHeadThreads) void given_budget_kernel(HeadArgs A) {
  if (blockIdx.z == 0) given_topk<kHeadThreads, 0, false, 1, true>(A);
  else gather_fixed<D, PAGED>(A, (int)blockIdx.z - 1);
}

typedef void (*GivenKernel)(HeadArgs);
GivenKernel given_budget_kernel_for(int d, bool paged) {
  if (d == 128) return paged ? given_budget_kernel<128, true> : given_budget_kernel<128, false>;
  return paged ? given_budget_kernel<64, true> : given_budget_kernel<64, false>;
}
// The instantiation for a head dimension (0: selection only) and cache layout.
template <int PHASE>
GivenKernel given_kernel_for(int d, bool paged) {
  if (d == 0) return given_topk_kernel<kHeadThreads, 0, false, PHASE>;
  if (d == 128) return paged ? given_topk_kernel<kHeadThreads, 128, true, PHASE> : given_topk_kernel<kHeadThreads, 128, false, PHASE>;
  return paged ? given_topk_kernel<kHeadThreads, 64, true, PHASE> : given_topk_kernel<kHeadThreads, 64, false, PHASE>;
}
GivenKernel given_kernel_for(int phase, int d, bool paged) {
  return phase == 0 ? given_kernel_for<0>(d, paged) : given_kernel_for<1>(d, paged);
}

}  // namespace

hipError_t set_given_kernel_attributes(const Plan& pl) {
  (void)pl;
  const int cap = 160 * 1024 - (int)head_kernel_static_lds_bytes();
  for (const int phase : {0, 1})
    for (const int d : {0, 64, 128})
      for (const bool paged : {false, true}) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(given_kernel_for(phase, d, paged)),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, cap);
        if (e != hipSuccess) return e;
      }
  for (const int d : {64, 128})
    for (const bool paged : {false, true}) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(given_budget_kernel_for(d, paged)),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, cap);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_given_select(const Plan& pl, const int32_t* seq_lens, const uint64_t* seq_seeds,
                               const int32_t* given_idx, const int32_t* given_cnt, const void* rcache, void* ws,
                               int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                               hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  A.given_idx = given_idx;
  A.given_cnt = given_cnt;
  A.rcache = rcache;
  A.rc = cache_layout(pl);
  const size_t lds = sizeof(uint32_t) * sampler_lds<kHeadThreads>(pl.p.n_max).end;
  hipLaunchKernelGGL(given_kernel_for(0, 0, false), dim3(pl.p.n_q_heads, pl.vbatch), dim3(kHeadThreads), lds, st, A);
  return hipGetLastError();
}

hipError_t launch_given_budget(const Plan& pl, const void* v, const int32_t* block_table, const int32_t* seq_lens,
                               const uint64_t* seq_seeds, void* ws, int32_t* out_idx, int32_t* out_counts, double* out_budget_raw,
                               float* out_stats, hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  A.v = static_cast<const uint16_t*>(v);
  A.L = pl.kv_v;
  A.L.block_table = block_table;
  A.part = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_gather_part);
  A.splits = given_fixed_splits(pl);
  A.part_slots = given_part_slots(pl);
  const size_t lds = sizeof(uint32_t) * sampler_lds<kHeadThreads>(pl.p.n_max).end;
  const GivenKernel kernel = A.splits > 0 ? given_budget_kernel_for(pl.p.head_dim, pl.p.kv_layout == VATT_LAYOUT_PAGED) : given_kernel_for(1, 0, false);
  hipLaunchKernelGGL(kernel, dim3(pl.p.n_q_heads, pl.vbatch, 1 + A.splits), dim3(kHeadThreads), lds, st, A);
  return hipGetLastError();
}

// Dynamic LDS of the selection phases of the caller-supplied-top-k path with scores / gather fused in: the first
// phase keeps its run of I_f and its share of the base sample (tokens and cache slots), the second its share of
// the final sample and the cross-wave sums.
int given_glist_cap(const Plan& pl, int splits) { return (pl.p.sink + pl.p.window + pl.k_max) / splits + 2; }
size_t given_fused_lds_bytes(const Plan& pl, int splits) {
  const size_t dl = (size_t)fused_dlist_cap(pl, splits);
  const size_t first = ((size_t)given_glist_cap(pl, splits) + 2 * dl) * sizeof(uint32_t);
  const size_t second = dl * sizeof(uint32_t) + (size_t)(kHeadThreads / kWave) * (pl.p.head_dim + 2) * sizeof(float);
  return sizeof(uint32_t) * head_lds<kHeadThreads, true>(pl.p.n_max).lists + std::max(first, second);
}

bool given_fused_fits(const Plan& pl, int splits) {
  if (splits < 1 || splits > 16 || (splits & (splits - 1)) != 0) return false;
  if (pl.p.target != VATT_TARGET_D || (pl.p.head_dim != 64 && pl.p.head_dim != 128)) return false;
  return given_fused_lds_bytes(pl, splits) + head_kernel_static_lds_bytes() <= 160 * 1024;
}

// The plan's own choice: as for the scored path, when there are at most half as many heads as compute units; and one
// workgroup per head when most compute units get one (whole step, us, separate kernels -> fused: 256 heads of 300 / 4K / 9K
// tokens 34.7 -> 31.1, 37.9 -> 35.9, 42.4 -> 40.3, of 4K with 64 columns 38.5 -> 34.1; 160 heads of 1K 31.7 both ways, of 6K with 5
// query tokens 40.4 -> 43.1).  That is with budgets near the base sample's size: 256 heads of 7K ragged at epsilon 0.05 / 0.03 /
// 0.02 / 0.01 36.8 / 42.2 / 56.7 / 70.3 apart, 35.2 / 43.5 / 59.3 / 92.4 fused.
int given_fused_splits_for(const Plan& pl) {
  const int heads = pl.vbatch * pl.p.n_q_heads;
  if (heads * 2 > pl.num_cus) return heads <= pl.num_cus && 4 * heads > 3 * pl.num_cus && given_fused_fits(pl, 1) ? 1 : 0;
  int s2 = 1;
  while (s2 * 2 * heads <= pl.num_cus && s2 < 16) s2 *= 2;
  while (s2 >= 1 && !given_fused_fits(pl, s2)) s2 /= 2;  // (fewer workgroups per head need longer LDS lists)
  return given_fused_fits(pl, s2) ? s2 : 0;
}

hipError_t launch_given_fused(const Plan& pl, int phase, const void* q, const void* k, const void* v,
                              const int32_t* block_table, const int32_t* seq_lens, const uint64_t* seq_seeds,
                              const int32_t* given_idx, const int32_t* given_cnt, const void* rcache, void* ws,
                              int32_t* out_idx, int32_t* out_counts, double* out_budget_raw, float* out_stats,
                              hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  // the final sample's first batch of draws passes from the first phase to the second
  static_assert(kHeadThreads == 2 * kPreThreads, "a thread's draws each");
  A.pre_tok = reinterpret_cast<uint4*>(static_cast<char*>(ws) + pl.off_pre_tok);
  A.pre_flags = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pl.off_pre_flags);
  const int S = pl.given_fuse_splits;
  A.given_idx = given_idx;
  A.given_cnt = given_cnt;
  A.rcache = rcache;
  A.rc = cache_layout(pl);
  A.glist_cap = given_glist_cap(pl, S);
  A.v = static_cast<const uint16_t*>(v);
  A.L = pl.kv_v;
  A.L.block_table = block_table;
  A.gq = static_cast<const uint16_t*>(q);
  A.gk = static_cast<const uint16_t*>(k);
  A.Lk = pl.kv_k;
  A.Lk.block_table = block_table;
  A.sm_scale = pl.sm_scale;
  A.part = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_gather_part);
  A.splits = S;
  A.split_shift = 0;
  while ((1 << A.split_shift) < S) ++A.split_shift;
  A.dlist_cap = fused_dlist_cap(pl, S);
  const dim3 grid(pl.p.n_q_heads, pl.vbatch, S);
  const size_t lds = given_fused_lds_bytes(pl, S);  // (the larger of the two phases' needs)
  const bool paged = pl.p.kv_layout == VATT_LAYOUT_PAGED;
  hipLaunchKernelGGL(given_kernel_for(phase, pl.p.head_dim, paged), grid, dim3(kHeadThreads), lds, st, A);
  return hipGetLastError();
}

}  // namespace vatt
