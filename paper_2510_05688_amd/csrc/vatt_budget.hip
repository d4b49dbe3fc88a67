// Budget and final sample of the targets N and SDPA (Algorithm 2 and the last draw of Algorithm 1), between the V-side statistics
// and the gather.
#include "vatt_select.h"

namespace vatt {
namespace {

// Targets N and SDPA, behind the V-side statistics: budget and final sample of every head (Algorithm 2; Algorithm 1, final
// sample).  The weights are those of the lists that phase 1 left, and so is the top-k bitmap.  D_f and N_f stay for the merge:
// the gather then reads the rows of the final sample only.
// What bounds it: one chain per head.  Everything that the budget waits for is asked for ahead of the first batch of draws, which
// is as large as the workgroup can make it: budgets of these targets go well beyond the base sample.
// Whole call, us, before (the selection kernel with its top-k step left out, then a gather of all listed rows) and now (this kernel, the
// gather of the final sample alone, and with few heads two workgroups each in phase 1, PRE): 4 x 16K tokens 87.6 -> 80.2, 16 x 32K
// 375 -> 359, 32 x 8K 328 -> 313, 4 x 128K 350 -> 325, 8 x 4K paged 83.3 -> 80.7, 2 x 9K of 16 heads 50.9 -> 47.5, one of 2K 34.5 -> 30.5.
// PRE: the first batch of draws comes from the second workgroups of phase 1.
template <int NT, bool OPTIONS, bool PRE>
__global__ __launch_bounds__(NT, 4) void budget_kernel(HeadArgs A) {
  touch_args<HeadArgs>();
  if constexpr (!OPTIONS) {
    A.nested = A.ascending = A.small_batches = 0;
    A.range_factor = 0.0;
    A.b_multiple = 1;
  }
  using O = HeadOps<NT>;
  extern __shared__ __align__(16) unsigned char dyn_smem[];
  typename O::HeadSmem& sm = *reinterpret_cast<typename O::HeadSmem*>(dyn_smem);
  const SamplerLds at = sampler_lds<NT>(A.n_max);
  uint32_t* lds = reinterpret_cast<uint32_t*>(dyn_smem);
  uint32_t* bm_f = lds + at.bm_f;
  const int h = head_of_block((int)blockIdx.x, A.Hq, A.Hkv, A.group_major), b = blockIdx.y;
  const int bh = b * A.Hq + h, tid = threadIdx.x;
  const int seq = seq_of_pair(b, A.q_len);
  // everything that can be asked for before the sizes are known
  const int n = A.head_rec[bh].n;
  const float m = A.head_rec[bh].m;
  const uint64_t seed = A.seq_seeds[seq];
  uint4 pre_t = make_uint4(0u, 0u, 0u, 0u);
  uint32_t pre_f = 0u;
  if constexpr (PRE) {
    pre_t = A.pre_tok[(int64_t)bh * NT + tid];
    pre_f = A.pre_flags[(int64_t)bh * NT + tid];
  }
  int32_t* c = A.out_counts + (int64_t)bh * 8;
  int flags = c[7];
  int32_t* idx = A.out_idx + (int64_t)bh * A.idx_cap;
  // (list entries of the first two rounds, whatever the lists hold: no list is longer than what follows its start)
  constexpr int U = 2;
  const int64_t last = A.idx_cap - 1;
  int top[U], base[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    top[u] = idx[min(A.seg_topk + u * NT + tid, last)];
    base[u] = idx[min(A.seg_base + u * NT + tid, last)];
  }
  // Numerator statistics from the V pass, per split {N_f[d], R1[d], R2, pad}: a thread per column, and one per split for R2.
  const int d = A.head_dim, stride = 2 * d + 2;
  const double* vp = A.vstat_part + (int64_t)bh * A.vstat_splits * stride;
  constexpr int VS = 8;
  double x[VS], y[VS], nf = 0.0, r1 = 0.0, r2 = 0.0;
  auto ask = [&](int s0) {
#pragma unroll
    for (int u = 0; u < VS; ++u) {
      const int from = min(s0 + u, A.vstat_splits - 1) * stride + tid;
      x[u] = vp[from];
      y[u] = vp[from + d];
    }
  };
  auto take = [&](int s0) {
#pragma unroll
    for (int u = 0; u < VS; ++u) {
      nf += s0 + u < A.vstat_splits ? x[u] : 0.0;
      r1 += s0 + u < A.vstat_splits ? y[u] : 0.0;
    }
  };
  if (tid < d) ask(0);
  else if (tid - d < A.vstat_splits) r2 = vp[(tid - d) * stride + 2 * d];  // (at most 32)
  for (int w = tid; w < 3 * (bitmap_words(A.n_max) / 4); w += NT)
    reinterpret_cast<uint4*>(bm_f)[w] = make_uint4(0u, 0u, 0u, 0u);  // the three bitmaps follow each other
  const HeadSizes hs = head_sizes(n, A.sp);
  const float* row = A.scores + (int64_t)bh * A.n_pad;
  // scores of the listed tokens, -inf where a thread has none (exp(-inf) = 0)
  const int n_base = hs.n_s > 0 ? hs.b0 : 0;
  float sc_top[U], sc_base[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    top[u] = min(max(top[u], 0), n - 1);
    sc_top[u] = row[top[u]];
    sc_base[u] = row[min(max(base[u], 0), n - 1)];
  }
  const float sc_sink = row[min(tid, n - 1)], sc_win = row[min(hs.mid_hi + tid, n - 1)];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u * NT + tid < hs.k) O::mark_bit(bm_f, (uint32_t)top[u]);
  for (int t = tid + U * NT; t < hs.k; t += NT) O::mark_bit(bm_f, (uint32_t)O::list_tok(idx, A.seg_topk + t, n));
  if (tid < d) {
    take(0);
    if (A.vstat_splits > VS) ask(VS);
  }

  typename O::Sampler S;
  S.taken = lds + at.taken;
  S.scratch = lds + at.scratch;
  S.mail = lds + at.mail;
  S.bm_f = bm_f;
  S.wpre = lds + at.wpre;
  S.row = row;
  S.seed = seed;
  S.stream = 1u;
  S.head = (uint32_t)h;
  S.query = (uint32_t)(b - seq * A.q_len);
  S.L = (uint32_t)max(hs.mid_hi - hs.mid_lo, 1);
  S.thr = (0u - S.L) % S.L;  // 2^32 mod L
  {
    const uint64_t dflt = 64ull * (uint64_t)S.L + 4096ull;
    S.cap = (uint32_t)min(A.draw_cap ? (uint64_t)A.draw_cap : dflt, 0x80000000ull);
  }
  S.m = m;
  S.dbg = nullptr;
  DrawBatch spec = {};
  const int plan_batch = ahead_blocks<NT>(A.small_batches, hs, final_draws(hs));
  const int first_batch = OPTIONS ? plan_batch : budget_blocks<NT>(hs);
  const bool want = hs.n_s > 0 && !A.nested;  // (a nested final sample rarely draws at all)
  if (want && PRE) {
    spec.blocks = first_batch;
    spec.ok = pre_ok(pre_f);
    spec.first = pre_first(pre_f);
    const uint32_t tk[4] = {pre_t.x, pre_t.y, pre_t.z, pre_t.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      spec.tok[e] = min(max(tk[e], (uint32_t)hs.mid_lo), (uint32_t)max(hs.mid_hi - 1, hs.mid_lo));
      if ((spec.ok >> e) & 1u) O::mark_bit(S.taken, spec.tok[e]);
    }
  } else if (want) {
    O::make_batch(spec, S, hs, 0u, first_batch, false, false, sm, tid);
  }
  constexpr bool kPlace = NT >= 1024;  // (as in the selection-only kernel)
  if (want && kPlace && A.splits == 1) {  // (else the second workgroup of phase 1 has left them)
#pragma unroll
    for (int e = 0; e < 4; ++e) spec.sc[e] = row[min(spec.tok[e], (uint32_t)(n - 1))];
    spec.have_sc = true;
  }

  double sums[3] = {0.0, 0.0, 0.0};  // D_f, and the base sample's weights and their squares
  auto fixed = [&](float sc) { sums[0] += (double)__expf(sc - m); };
  auto sampled = [&](float sc) {
    const double w = (double)__expf(sc - m);
    sums[1] += w;
    sums[2] += w * w;
  };
#pragma unroll
  for (int u = 0; u < U; ++u) {
    fixed(u * NT + tid < hs.k ? sc_top[u] : -INFINITY);
    sampled(u * NT + tid < n_base ? sc_base[u] : -INFINITY);
  }
  for (int t = tid + U * NT; t < hs.k; t += NT) fixed(row[O::list_tok(idx, A.seg_topk + t, n)]);
  for (int t = tid + U * NT; t < n_base; t += NT) sampled(row[O::list_tok(idx, A.seg_base + t, n)]);
  fixed(tid < hs.n_sink ? sc_sink : -INFINITY);
  fixed(tid < hs.n_win ? sc_win : -INFINITY);
  for (int i = tid + NT; i < hs.n_sink; i += NT) fixed(row[i]);
  for (int i = tid + NT; i < hs.n_win; i += NT) fixed(row[hs.mid_hi + i]);
  O::block_sum(sums, sm);
  const double D_f = sums[0];
  double* fixed_sums = A.fixed_sums + (int64_t)bh * kFixedStride;  // (this workgroup has read the head's flags)
  if (tid < d) {
    if (A.vstat_splits > VS) take(VS);
    for (int s0 = 2 * VS; s0 < A.vstat_splits; s0 += VS) {
      ask(s0);
      take(s0);
    }
    fixed_sums[1 + tid] = nf;
  }
  if (tid == 0) fixed_sums[0] = D_f;
  double sigma2 = 0.0, b_star = 0.0, tr_sigma = 0.0, nhat_sq = 0.0, D_hat = D_f;
  int bfin = 0;
  if (hs.n_s > 0) {
    const double ns = (double)hs.n_s;
    const double nh = nf + ns * r1 / (double)hs.b0;
    double t3[3] = {nh * nh, r1 * r1, r2};  // (zero where a thread has no column)
    O::block_sum(t3, sm);
    nhat_sq = t3[0];
    const double rho_N = numerator_rho(hs.n_s, hs.b0, t3[1], t3[2], nhat_sq, &tr_sigma);
    const Budget bud = algorithm2_budget(A, hs.n_s, hs.b0, D_f, sums[1], sums[2], rho_N, 1.0);
    sigma2 = bud.sigma2;
    b_star = bud.b_star;
    bfin = bud.b;
    D_hat = bud.D_hat;
  }
  if (tid == 0 && A.out_stats) {
    float* st = A.out_stats + (int64_t)bh * 4;
    st[0] = (float)D_hat;
    st[1] = (float)sigma2;
    st[2] = (float)tr_sigma;
    st[3] = (float)nhat_sq;
  }

  // ---- I_dyn (Algorithm 1, final sample) ----
  bool dyn_placed = false;
  if (bfin > 0) {
    Emit E = emit_to(idx + A.seg_dyn, (uint32_t)A.b_max);
    if (kPlace) E.sc_dst = A.place_sc + (int64_t)bh * A.idx_cap + A.seg_dyn;
    // (the flag of further batches goes by the size that the first batch has elsewhere)
    const int f = A.nested ? O::draw_nested(S, hs, (uint32_t)hs.b0, (uint32_t)bfin, bm_f, idx + A.seg_base, idx + A.seg_dyn,
                                            (uint32_t)A.b_max, A.small_batches, sm)
                           : O::draw_sample(S, hs, (uint32_t)bfin, spec, want, A.small_batches, E, nullptr, nullptr, sm, 0u, 0u,
                                            !OPTIONS, plan_batch);
    flags |= ((f & 1) ? kFlagDynComplement : 0) | ((f & 2) ? kFlagDynBatches : 0) | ((f & 4) ? kFlagDrawCap : 0);
    // (one batch made ahead with its scores held the whole sample, and the list stays in acceptance order)
    dyn_placed = kPlace && !A.nested && !A.ascending && want && f == 0;
    if (A.ascending && !A.nested && !(f & 1))
      O::sort_ascending(idx + A.seg_dyn, (uint32_t)min(bfin, A.b_max), S.scratch, S.wpre, n, sm);
  }
  if (tid == 0) {
    c[0] = hs.n_sink;
    c[1] = hs.n_win;
    c[2] = hs.k;
    c[3] = hs.n_s > 0 ? hs.b0 : 0;
    c[4] = bfin;
    c[5] = hs.n_s;
    c[6] = n;
    c[7] = flags;
    if (A.out_budget_raw) A.out_budget_raw[bh] = b_star;
    HeadRec& r = A.head_rec[bh];  // (the rest stays as phase 1 has written it: a copy of it went through scratch memory, 0.5 us of the call)
    r.scale = bfin > 0 ? (float)((double)hs.n_s / (double)bfin) : 0.f;
    r.b = bfin;
    r.b_keep = (A.nested && bfin > 0) ? hs.b0 : 0;
    r.tail_by_token = dyn_placed ? 0 : 1;
  }
}

typedef void (*BudgetKernel)(HeadArgs);
BudgetKernel budget_kernel_for(int threads, bool options, bool pre) {
  if (threads == kHeadThreadsLong) return options ? budget_kernel<kHeadThreadsLong, true, false> : budget_kernel<kHeadThreadsLong, false, false>;
  if (options) return budget_kernel<kHeadThreads, true, false>;
  return pre ? budget_kernel<kHeadThreads, false, true> : budget_kernel<kHeadThreads, false, false>;
}

}  // namespace

hipError_t set_budget_kernel_attributes() {
  // (as for the selection kernels: the limit belongs to the kernel, so it is raised to all a CU has)
  for (const int threads : {kHeadThreads, kHeadThreadsLong})
    for (const bool options : {false, true})
      for (const bool pre : {false, true}) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(budget_kernel_for(threads, options, pre)),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

hipError_t launch_budget(const Plan& pl, const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws, int32_t* out_idx,
                         int32_t* out_counts, double* out_budget_raw, float* out_stats, hipStream_t st) {
  HeadArgs A;
  fill_head_args(A, pl, seq_lens, seq_seeds, ws, out_idx, out_counts, out_budget_raw, out_stats);
  const vatt_params& p = pl.p;
  const int threads = pl.head_threads;
  A.splits = head_pair(pl, 1) ? 2 : 1;
  A.pre_tok = reinterpret_cast<uint4*>(static_cast<char*>(ws) + pl.off_pre_tok);
  A.pre_flags = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pl.off_pre_flags);
  const size_t lds = sizeof(uint32_t) * (threads == kHeadThreadsLong ? sampler_lds<kHeadThreadsLong>(p.n_max) : sampler_lds<kHeadThreads>(p.n_max)).end;
  hipLaunchKernelGGL(budget_kernel_for(threads, head_options(pl), A.splits == 2), dim3(p.n_q_heads, pl.vbatch), dim3(threads), lds, st, A);
  return hipGetLastError();
}

}  // namespace vatt
