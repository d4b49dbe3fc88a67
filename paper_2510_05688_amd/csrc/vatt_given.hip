// Decode step with a caller-supplied top-k set (the paper's pred-top-index hook, Section 4.1: any approximate
// top-k method may supply I_t): no pass over the whole K cache.  Scores exist only for the tokens that are
// attended:
//
//   sparse_score_kernel   s_i = sm_scale * <K[i], q> for the tokens of I_f and I_bs, written next to their
//                         places in the index lists
//   given_gather_kernel   the N and D sums of Section 4.1 over [I_f, I_dyn]: scores of I_f from the sparse
//                         list, scores of I_dyn computed here from their K rows (with nested samples the
//                         base-sample part of I_dyn has its scores in the list already); V rows gathered as
//                         in the dense-scored path.  No head maximum is known in advance, so every wave keeps a
//                         running maximum and rescales (online softmax), and the merge combines the splits'
//                         (max, D, N) partials the same way.
//
// grid = (query heads, splits, sequences) for both, head fastest and in head_of_block order: the splits of a
// head, and the heads of a KV head, then share an XCD and its L2 (index lists, and the K and V rows they have in
// common); d/8 adjacent lanes read one K or V row with one 16-byte load each.  Of a head's splits only as many take
// part as its list has steps for (used_splits).
//
// What bounds them: the chain record -> list entry -> row on short lists, the pace of 256-byte rows in no order (about 6 TB/s)
// on long ones.  Whole step, us, before (every lane of a row worked out its place, its entry requested when its step came, a
// maximum per lane group, all splits busy) and after: 16 x 32K tokens 127 -> 119.5, 16 x 4K 71.5 -> 50.4, 8 x 0.5K - 7K
// paged 59 -> 42, 32 x 1.5K paged 97 -> 78, 1 x 9K with 16 query tokens 89 -> 72.5, 24 x 8K of 64 columns 73.7 -> 46.
#include <type_traits>

#include "vatt_internal.h"

namespace vatt {
namespace {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc,
                                         false);
}

struct GivenArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  KVLayout Lk, Lv;
  const HeadRec* head_rec;
  const int32_t* idx;
  float* sparse;      // [B*Hq][idx_cap]: score of the token at the same place of the index lists
  float* part;        // [B*Hq][splits][d + 4]: N[d], D, running maximum
  float* vstat;       // [B*Hq][splits][2d + 4]: N_f[d], R1[d], R2, maximum (numerator statistics, targets N / SDPA)
  float* out_o;
  float* out_lse;
  // (the sink segment starts at place 0: with a field of its own, what the score kernels read goes on into a further line of arguments,
  // 0.5 us of the short calls)
  int64_t seg_win, seg_topk, seg_base, seg_dyn, idx_cap;
  int Hq, group, splits;
  int part_slots, first_slot;  // partial sums of a head in all; the first of the gather's
  int group_major;  // see head_of_block (the KV head count is Hq / group)
  int q_len;  // query tokens per sequence: blockIdx.z = sequence * q_len + query token
  float sm_scale;
  // random cache of base-sample rows: heads whose HeadRec.base_cached is set read their base sample's rows from it
  const void* rcache;
  CacheLayout rc;
  const int32_t* base_slot;  // [B*Hq][b0_max]
  int b0_max;
};

template <int D>
__device__ __forceinline__ void load_q(const GivenArgs& A, int bh, int sub, uint32_t (&qw)[4]) {
  const uint4 t = *reinterpret_cast<const uint4*>(A.q + (int64_t)bh * D + sub * 8);
  qw[0] = t.x;
  qw[1] = t.y;
  qw[2] = t.z;
  qw[3] = t.w;
}

template <int LPR>
__device__ __forceinline__ float row_score(const uint4& kv, const uint32_t (&qw)[4], float sm_scale) {
  float a = 0.f;
  a = dot2_bf16(kv.x, qw[0], a);
  a = dot2_bf16(kv.y, qw[1], a);
  a = dot2_bf16(kv.z, qw[2], a);
  a = dot2_bf16(kv.w, qw[3], a);
  return group_sum<LPR>(a) * sm_scale + 0.0f;
}

// Scores of the tokens of I_f and I_bs (HeadRec.b holds |I_bs| at this point), without the numerator statistics.  What
// belongs to a row (list place, token, slot of the random cache) is done by the row's own lane, as in gather_kernel, and
// the list entry of the next step is requested one step ahead; row and score change lanes by wave shuffles.
template <int D, bool PAGED>
__global__ __launch_bounds__(kGatherThreads, 8) void sparse_score_kernel(GivenArgs A) {
  constexpr int LPR = D / 8;
  constexpr int RPW = kWave / LPR;
  constexpr int WAVES = kGatherThreads / kWave;
  constexpr int RPB = RPW * WAVES;
  constexpr int U = 8;
  static_assert(U <= LPR && RPW * U <= kWave, "a lane per row of a step, and one per row of a lane group");
  const int h = head_of_block((int)blockIdx.x, A.Hq, div_group(A.Hq, A.group), A.group_major), split = blockIdx.y, b = blockIdx.z;
  const int bh = b * A.Hq + h;
  const int kvh = div_group(h, A.group), seq = seq_of_pair(b, A.q_len);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rsub = lane / LPR;
  const HeadRec r = A.head_rec[bh];
  uint32_t qw[4];
  load_q<D>(A, bh, sub, qw);
  const int total = r.n_sink + r.n_win + r.k + r.b;
  const int splits = used_splits(A.splits, total, RPB * U);
  if (split >= splits) return;
  const bool shared_rows = rows_are_shared(total, A.group_major ? A.q_len * A.group : A.q_len, r.n);
  const int per = (total + splits - 1) / splits;
  const int p_lo = split * per, p_hi = min(p_lo + per, total);
  const int32_t* idx = A.idx + (int64_t)bh * A.idx_cap;
  float* sp = A.sparse + (int64_t)bh * A.idx_cap;
  const bool cached = r.base_cached != 0;
  const uint16_t* cache_k = cached ? reinterpret_cast<const uint16_t*>(cache_record(A.rcache, A.rc, seq, div_group(A.Hq, A.group), kvh) + A.rc.off_k) : nullptr;
  const int32_t* slots_of = A.base_slot + (int64_t)bh * A.b0_max;
  const uint16_t* k_head = PAGED ? A.k : A.k + (int64_t)seq * A.Lk.seq_stride + (int64_t)kvh * A.Lk.head_stride;
  const int n_sw = r.n_sink + r.n_win, n_fix = n_sw + r.k;
  const uint32_t seg_win = (uint32_t)A.seg_win, seg_topk = (uint32_t)A.seg_topk;
  const uint32_t seg_base = (uint32_t)A.seg_base;
  const int mine = (lane / RPW) * RPB + wave * RPW + lane % RPW;  // the row of a step that this lane prepares
  auto place_of = [&](int p0) {
    const int pc = min(p0 + mine, p_hi - 1), t2 = pc - n_sw, t3 = pc - n_fix;
    const uint32_t edge = pc < r.n_sink ? (uint32_t)pc : seg_win + (uint32_t)(pc - r.n_sink);
    return t3 >= 0 ? seg_base + (uint32_t)t3 : t2 >= 0 ? seg_topk + (uint32_t)t2 : edge;
  };
  // a row in the cache is known by its slot, with the top bit set
  auto entry_of = [&](uint32_t place) {
    return cached && place >= seg_base ? slots_of[place - seg_base] | (int)0x80000000 : idx[place];
  };
  uint32_t place_next = 0;
  int entry_next = 0;
  if (p_lo < p_hi) entry_next = entry_of(place_next = place_of(p_lo));
  // (the loop twice, one for each kind of load: with the choice inside it took 15 registers and a wave per SIMD more)
  auto walk = [&](auto load) {
    for (int p0 = p_lo; p0 < p_hi; p0 += RPB * U) {
      const uint32_t place = place_next;
      const int entry = entry_next;
      entry_next = entry_of(place_next = place_of(p0 + RPB * U));  // (beyond the range: its last place once more)
      const bool in_cache = cached && entry < 0;
      const int row_mine = in_cache ? min(entry & 0x7fffffff, A.rc.slots - 1) | (int)0x80000000 : min(max(entry, 0), r.n - 1);
      int row[U], blk[U];
      uint4 kv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) row[u] = __shfl(row_mine, u * RPW + rsub);
#pragma unroll
      for (int u = 0; u < U; ++u) blk[u] = kv_block<PAGED>(A.Lk, seq, row[u] < 0 ? 0 : row[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = row[u] & 0x7fffffff;
        const uint16_t* at = PAGED ? A.k + kv_row_offset_in<true>(A.Lk, seq, kvh, i, blk[u]) : k_head + (uint32_t)i * (uint32_t)D;
        // (rows of the cache without the non-temporal hint: the group's heads share them; 115.7 -> 110.7 us for a whole step of
        // 16 x 32K tokens)
        if (row[u] < 0) kv[u] = *reinterpret_cast<const uint4*>(cache_k + ((uint32_t)i * (uint32_t)D + (uint32_t)(sub * 8)));
        else kv[u] = load(at + sub * 8);
      }
      __builtin_amdgcn_sched_barrier(0);
      float s = 0.f;  // lane u of a group keeps the score of the group's row u
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float su = row_score<LPR>(kv[u], qw, A.sm_scale);
        s = sub == u ? su : s;
      }
      const int from = (sub % U) * RPW + rsub;  // the lane that prepared that row
      const uint32_t to = (uint32_t)__shfl((int)place, from);
      if (sub < U && p0 + sub * RPB + wave * RPW + rsub < p_hi) sp[to] = s;
    }
  };
  if (shared_rows) walk(LoadShared{});
  else walk(LoadOnce{});
}

// The same with the numerator statistics (targets N and SDPA): the V rows of the same tokens are read as well and the
// statistics of Algorithm 2 are accumulated on the way: N_f = sum_{I_f} w V, R1 = sum_{I_bs} w V, R2 = sum_{I_bs} ||w V||^2 with
// w = exp(s - max); no maximum is known yet, so every lane group keeps a running one and rescales.
template <int D, bool PAGED>
__global__ __launch_bounds__(kGatherThreads) void sparse_stats_kernel(GivenArgs A) {
  constexpr int LPR = D / 8;
  constexpr int RPW = kWave / LPR;
  constexpr int WAVES = kGatherThreads / kWave;
  constexpr int RPB = RPW * WAVES;
  constexpr int GROUPS = RPB;
  constexpr int U = 8;
  const int h = head_of_block((int)blockIdx.x, A.Hq, div_group(A.Hq, A.group), A.group_major), split = blockIdx.y, b = blockIdx.z;
  const int bh = b * A.Hq + h;
  const int kvh = div_group(h, A.group);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, rsub = lane / LPR;
  const HeadRec r = A.head_rec[bh];
  const int32_t* idx = A.idx + (int64_t)bh * A.idx_cap;
  float* sp = A.sparse + (int64_t)bh * A.idx_cap;
  const int total = r.n_sink + r.n_win + r.k + r.b;
  const int per = (total + A.splits - 1) / A.splits;
  const int p_lo = split * per, p_hi = min(p_lo + per, total);
  const unsigned char* cache_rec = r.base_cached ? cache_record(A.rcache, A.rc, seq_of_pair(b, A.q_len), div_group(A.Hq, A.group), kvh) : nullptr;
  const int32_t* slots_of = A.base_slot + (int64_t)bh * A.b0_max;
  uint32_t qw[4];
  load_q<D>(A, bh, sub, qw);
  float acc_f[8], acc_b[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc_f[c] = acc_b[c] = 0.f;
  float r2 = 0.f, m_run = -INFINITY;
  // U rows per lane group at a time, without a branch per row: places in the lists (arithmetic), tokens (one
  // load each; for a base sample that came from the random cache also its slots), rows (one or two loads each),
  // then the arithmetic.  A slot beyond the range repeats the range's last row and writes nothing.  The base
  // sample has its own walk: its rows may come from the cache, and its statistics go to sums of their own.
  const int n_fix = r.n_sink + r.n_win + r.k;
  const bool cached = r.base_cached != 0;
  auto walk = [&](int lo, int hi, auto tail_tag) {
    constexpr bool kTail = decltype(tail_tag)::value;
    for (int p0 = lo + wave * RPW + rsub; p0 < hi; p0 += RPB * U) {
      int64_t place[U];
      bool valid[U];
      int tok[U], slot[U];
      uint4 kv[U], vv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * RPB;
        valid[u] = p < hi;
        const int pc = min(p, hi - 1);
        place[u] = kTail ? A.seg_base + (pc - n_fix)
                         : fixed_place(pc, r.n_sink, r.n_win, 0, A.seg_win, A.seg_topk);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        tok[u] = idx[place[u]];
        slot[u] = 0;
      }
      if (kTail && cached) {
        // the copies of the rows in the cache: rows of neighbouring slots, shared by the group's heads
#pragma unroll
        for (int u = 0; u < U; ++u) slot[u] = slots_of[place[u] - A.seg_base];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t so = (int64_t)min(max(slot[u], 0), A.rc.slots - 1) * D + sub * 8;
          kv[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(cache_rec + A.rc.off_k) + so);
          vv[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(cache_rec + A.rc.off_v) + so);
        }
      } else {
        int blk[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          tok[u] = min(max(tok[u], 0), r.n - 1);
          blk[u] = kv_block<PAGED>(A.Lk, seq_of_pair(b, A.q_len), tok[u]);  // (K and V share the block table)
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          kv[u] = load_stream_16(A.k + kv_row_offset_in<PAGED>(A.Lk, seq_of_pair(b, A.q_len), kvh, tok[u], blk[u]) + sub * 8);
          vv[u] = load_stream_16(A.v + kv_row_offset_in<PAGED>(A.Lv, seq_of_pair(b, A.q_len), kvh, tok[u], blk[u]) + sub * 8);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float s = row_score<LPR>(kv[u], qw, A.sm_scale);
        if (valid[u] && sub == 0) sp[place[u]] = s;
        if (valid[u]) {
          if (s > m_run) {
            const float f = __expf(m_run - s);  // 0 when m_run is -inf
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              acc_f[c] *= f;
              acc_b[c] *= f;
            }
            r2 *= f * f;
            m_run = s;
          }
          const float wt = __expf(s - m_run);
          const uint32_t ww[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float x = wt * bf16_lo(ww[c]), y = wt * bf16_hi(ww[c]);
            if constexpr (kTail) {
              acc_b[2 * c] += x;
              acc_b[2 * c + 1] += y;
              r2 += x * x + y * y;
            } else {
              acc_f[2 * c] += x;
              acc_f[2 * c + 1] += y;
            }
          }
        }
      }
    }
  };
  walk(p_lo, min(p_hi, n_fix), std::false_type{});
  walk(max(p_lo, n_fix), p_hi, std::true_type{});
  // every lane group has its own (maximum, N_f, R1, R2 share): bring them to the workgroup's maximum and add
  __shared__ float s_f[GROUPS][D], s_b[GROUPS][D];
  __shared__ float s_r2[GROUPS][LPR], s_m[GROUPS];
  const int g = wave * RPW + rsub;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    s_f[g][sub * 8 + c] = acc_f[c];
    s_b[g][sub * 8 + c] = acc_b[c];
  }
  s_r2[g][sub] = r2;
  if (sub == 0) s_m[g] = m_run;
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int j = 0; j < GROUPS; ++j) M = fmaxf(M, s_m[j]);
  float* out = A.vstat + ((int64_t)bh * A.splits + split) * (2 * D + 4);
  if (tid < D) {
    float a = 0.f, c2 = 0.f;
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) {
      const float f = s_m[j] > -INFINITY ? __expf(s_m[j] - M) : 0.f;
      a += s_f[j][tid] * f;
      c2 += s_b[j][tid] * f;
    }
    out[tid] = a;
    out[D + tid] = c2;
  }
  if (tid == 0) {
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) {
      const float f = s_m[j] > -INFINITY ? __expf(s_m[j] - M) : 0.f;
      float q2 = 0.f;
#pragma unroll
      for (int c = 0; c < LPR; ++c) q2 += s_r2[j][c];
      t += q2 * f * f;
    }
    out[2 * D] = t;
    out[2 * D + 1] = M;
  }
}

// N and D over [I_f, I_dyn], or I_dyn alone where the sums over I_f are made beside the second selection phase, by list place, in the
// manner of gather_kernel: what belongs to a row is done by the row's own
// lane, list entries and known scores are requested one step ahead, all rows of a step are in flight together.  Rows of newly
// drawn tokens bring their K row along; lane u of a group keeps the score of the group's row u and passes it to the row's
// own lane.  A wave has one running maximum, raised once per step.
template <int D, bool PAGED, bool BESIDE>
__global__ __launch_bounds__(kGatherThreads) void given_gather_kernel(GivenArgs A) {
  constexpr int LPR = D / 8;
  constexpr int RPW = kWave / LPR;
  constexpr int WAVES = kGatherThreads / kWave;
  constexpr int RPB = RPW * WAVES;
  constexpr int U = 8;
  constexpr int ROWS_W = RPW * U;
  static_assert(U <= LPR && ROWS_W <= kWave, "a lane per row of a step, and one per row of a lane group");
  const int h = head_of_block((int)blockIdx.x, A.Hq, div_group(A.Hq, A.group), A.group_major), split = blockIdx.y, b = blockIdx.z;
  const int bh = b * A.Hq + h;
  const int kvh = div_group(h, A.group), seq = seq_of_pair(b, A.q_len);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, rsub = lane / LPR;
  const HeadRec r = A.head_rec[bh];
  uint32_t qw[4];
  load_q<D>(A, bh, sub, qw);
  const int n_fix = r.n_sink + r.n_win + r.k, total = n_fix + r.b;
  const int first = BESIDE ? n_fix : 0, count = total - first;
  const int splits = used_splits(A.splits, count, RPB * U);
  if (split >= splits) return;
  const bool shared_rows = rows_are_shared(total, A.group_major ? A.q_len * A.group : A.q_len, r.n, A.group_major && A.group > 1 ? 3 : 2);
  const int per = (count + splits - 1) / splits;
  const int p_lo = first + split * per, p_hi = min(p_lo + per, total);
  const int32_t* idx = A.idx + (int64_t)bh * A.idx_cap;
  const float* sp = A.sparse + (int64_t)bh * A.idx_cap;
  const uint16_t* k_head = PAGED ? A.k : A.k + (int64_t)seq * A.Lk.seq_stride + (int64_t)kvh * A.Lk.head_stride;
  const uint16_t* v_head = PAGED ? A.v : A.v + (int64_t)seq * A.Lv.seq_stride + (int64_t)kvh * A.Lv.head_stride;
  const float tail_bias = r.scale > 0.f ? __logf(r.scale) : 0.f;  // ln(n_s / b): sampled tokens weigh n_s / b
  const int n_sw = r.n_sink + r.n_win;
  const int n_kept = n_fix + min(max(r.b_keep, 0), r.b);  // (nested samples: these have their scores in the base sample's places)
  const uint32_t seg_win = (uint32_t)A.seg_win, seg_topk = (uint32_t)A.seg_topk;
  const uint32_t seg_base = (uint32_t)A.seg_base, seg_dyn = (uint32_t)A.seg_dyn;
  const int mine = (lane / RPW) * RPB + wave * RPW + lane % RPW;  // the row of a step that this lane prepares

  int entry_next = 0;
  float sc_next = 0.f;
  auto request = [&](int p0) {  // (beyond the range: its last place once more)
    const int pc = min(p0 + mine, p_hi - 1), t2 = pc - n_sw, t3 = pc - n_fix;
    const uint32_t edge = pc < r.n_sink ? (uint32_t)pc : seg_win + (uint32_t)(pc - r.n_sink);
    const uint32_t fixed = t2 >= 0 ? seg_topk + (uint32_t)t2 : edge;
    entry_next = idx[t3 >= 0 ? seg_dyn + (uint32_t)t3 : fixed];
    sc_next = pc < n_kept ? sp[t3 >= 0 ? seg_base + (uint32_t)t3 : fixed] : 0.f;
  };
  if (p_lo < p_hi) request(p_lo);

  float acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.f;
  float dsum = 0.f, m_run = -INFINITY;
  // (the loop twice, one for each kind of load: with the choice inside it took 15 registers and a wave per SIMD more)
  auto walk = [&](auto load) {
    for (int p0 = p_lo; p0 < p_hi; p0 += RPB * U) {
      const int p = p0 + mine;
      const bool valid = lane < ROWS_W && p < p_hi, tail = p >= n_fix, drawn = valid && p >= n_kept;
      const int tok_mine = min(max(entry_next, 0), r.n - 1);
      float sc = sc_next;
      request(p0 + RPB * U);
      int tok[U], blk[U];
      uint4 kv[U], vv[U];
      // (a row with its K row: the top bit of its token)
#pragma unroll
      for (int u = 0; u < U; ++u) tok[u] = __shfl(drawn ? tok_mine | (int)0x80000000 : tok_mine, u * RPW + rsub);
#pragma unroll
      for (int u = 0; u < U; ++u) blk[u] = kv_block<PAGED>(A.Lv, seq, tok[u] & 0x7fffffff);  // (K and V share the block table)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = tok[u] & 0x7fffffff;
        const int64_t o = PAGED ? kv_row_offset_in<true>(A.Lk, seq, kvh, i, blk[u]) : 0;
        kv[u] = make_uint4(0u, 0u, 0u, 0u);
        if (tok[u] < 0) kv[u] = load(PAGED ? A.k + o + sub * 8 : k_head + ((uint32_t)i * (uint32_t)D + (uint32_t)(sub * 8)));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = tok[u] & 0x7fffffff;
        const int64_t o = PAGED ? kv_row_offset_in<true>(A.Lv, seq, kvh, i, blk[u]) : 0;
        vv[u] = load(PAGED ? A.v + o + sub * 8 : v_head + ((uint32_t)i * (uint32_t)D + (uint32_t)(sub * 8)));
      }
      __builtin_amdgcn_sched_barrier(0);
      if (__any(drawn)) {
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float su = row_score<LPR>(kv[u], qw, A.sm_scale);
          s = sub == u ? su : s;
        }
        const float computed = __shfl(s, (lane % RPW) * LPR + (lane / RPW) % U);
        sc = drawn ? computed : sc;
      }
      const float e = valid ? sc + (tail ? tail_bias : 0.f) : -INFINITY;
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
      for (int u = 0; u < U; ++u) {
        const float wt = __shfl(wt_mine, u * RPW + rsub);
        const uint32_t ww[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          acc[2 * c] += wt * bf16_lo(ww[c]);
          acc[2 * c + 1] += wt * bf16_hi(ww[c]);
        }
      }
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
  float* part = A.part + ((int64_t)bh * A.part_slots + (BESIDE ? A.first_slot : 0) + split) * (D + 4);
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

// Combines the per-split (maximum, D, N) partials of a head in split order: O = N / D, lse = M + ln D.  APART: only the splits that took
// part (used_splits) have written theirs; the first fixed_splits are those of I_f beside the second selection phase, the others the
// gather's.  Bound by the trip to memory: the first 16 are requested beside the head record.
template <int D, bool APART, bool BESIDE>
__global__ __launch_bounds__(D) void given_merge_kernel(const float* __restrict__ part, const HeadRec* __restrict__ head_rec,
                                                        int splits, int Hq, float* __restrict__ out_o,
                                                        float* __restrict__ out_lse, int group_major, int Hkv, int fixed_splits,
                                                        int part_slots) {
  const int h = head_of_block((int)blockIdx.x, Hq, Hkv, group_major), b = blockIdx.y, bh = b * Hq + h;
  const int c = threadIdx.x;
  const float* p = part + (int64_t)bh * part_slots * (D + 4);
  // lane s of every wave: (D, maximum) of split s; all lanes: their column of the splits, eight at a time
  const float2 dm = *reinterpret_cast<const float2*>(p + min(c & (kWave - 1), splits - 1) * (D + 4) + D);
  constexpr int U = 8;
  float v[U], v2[U];
  auto load = [&](float (&to)[U], int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) to[u] = p[min(s0 + u, splits - 1) * (D + 4) + c];
  };
  load(v, 0);
  if (splits > U) load(v2, U);
  const int s = c & (kWave - 1);
  bool mine = s < splits;
  if constexpr (APART) {
    constexpr int step_rows = kGatherThreads / (D / 8) * 8;
    const HeadRec r = head_rec[bh];
    const int n_fix = r.n_sink + r.n_win + r.k;
    const int fixed = BESIDE ? fixed_splits : 0;
    mine = s < fixed ? s < used_splits(fixed, n_fix, fixed_step_rows(D))
                     : s - fixed < used_splits(splits - fixed, BESIDE ? r.b : n_fix + r.b, step_rows) && s < splits;
  }
  const uint64_t took_part = __ballot(mine);
  const float M = wave_max(mine ? dm.y : -INFINITY);
  // (a split with no score but NaN has the maximum -inf and hands its NaN on, times 0)
  const float f = mine && dm.y > -INFINITY ? __expf(dm.y - M) : 0.f, df = mine ? dm.x * f : 0.f;
  float a = 0.f, dtot = 0.f;
  auto add = [&](const float (&from)[U], int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float fu = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), s0 + u));
      a += (took_part >> (s0 + u)) & 1u ? from[u] * fu : 0.f;  // (what a split without a part left behind is not looked at)
      dtot += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(df), s0 + u));
    }
  };
  add(v, 0);
  if (took_part >> U) add(v2, U);
  for (int s0 = 2 * U; s0 < splits && took_part >> s0; s0 += U) {
    load(v, s0);
    add(v, s0);
  }
  out_o[(int64_t)bh * D + c] = a / dtot;
  if (c == 0 && out_lse) out_lse[bh] = M + logf(dtot);
}

template <int D>
auto given_gather_for(bool paged, bool beside) {
  if (paged) return beside ? given_gather_kernel<D, true, true> : given_gather_kernel<D, true, false>;
  return beside ? given_gather_kernel<D, false, true> : given_gather_kernel<D, false, false>;
}

template <int D>
hipError_t launch_given_d(const Plan& pl, int stage, const void* q, const void* k, const void* v,
                          const int32_t* block_table, const void* rcache, void* ws, const int32_t* out_idx,
                          float* out_o, float* out_lse, hipStream_t st) {
  const vatt_params& p = pl.p;
  char* w = static_cast<char*>(ws);
  GivenArgs A;
  A.q = static_cast<const uint16_t*>(q);
  A.k = static_cast<const uint16_t*>(k);
  A.v = static_cast<const uint16_t*>(v);
  A.Lk = pl.kv_k;
  A.Lk.block_table = block_table;
  A.Lv = pl.kv_v;
  A.Lv.block_table = block_table;
  A.head_rec = reinterpret_cast<const HeadRec*>(w + pl.off_head_rec);
  A.idx = out_idx;
  A.sparse = reinterpret_cast<float*>(w + pl.off_sparse);
  A.part = reinterpret_cast<float*>(w + pl.off_gather_part);
  A.vstat = reinterpret_cast<float*>(w + pl.off_vstat_part);
  A.out_o = out_o;
  A.out_lse = out_lse;
  A.seg_win = pl.seg_off[1];
  A.seg_topk = pl.seg_off[2];
  A.seg_base = pl.seg_off[3];
  A.seg_dyn = pl.seg_off[4];
  A.idx_cap = (int64_t)pl.idx_cap;
  A.Hq = p.n_q_heads;
  A.group = pl.group;
  A.splits = stage == 0 ? pl.given_splits : given_tail_splits(pl);
  A.first_slot = given_fixed_splits(pl);
  A.part_slots = A.first_slot > 0 ? given_part_slots(pl) : A.splits;
  A.q_len = pl.q_len;
  A.group_major = pl.group_major;
  A.sm_scale = pl.sm_scale;
  A.rcache = rcache;
  A.rc = cache_layout(pl);
  A.base_slot = reinterpret_cast<const int32_t*>(w + pl.off_base_slot);
  A.b0_max = pl.b0_max;
  const bool paged = p.kv_layout == VATT_LAYOUT_PAGED;
  const bool stats = p.target != VATT_TARGET_D;
  if (stage == 0 && !stats) A.splits = pl.sparse_splits;  // scores only: no partial sums, any number of workgroups
  dim3 grid(p.n_q_heads, A.splits, pl.vbatch);
  if (stage == 0) {
    if (paged && stats) hipLaunchKernelGGL((sparse_stats_kernel<D, true>), grid, dim3(kGatherThreads), 0, st, A);
    else if (paged) hipLaunchKernelGGL((sparse_score_kernel<D, true>), grid, dim3(kGatherThreads), 0, st, A);
    else if (stats) hipLaunchKernelGGL((sparse_stats_kernel<D, false>), grid, dim3(kGatherThreads), 0, st, A);
    else hipLaunchKernelGGL((sparse_score_kernel<D, false>), grid, dim3(kGatherThreads), 0, st, A);
    return hipGetLastError();
  }
  const bool beside = A.first_slot > 0;
  hipLaunchKernelGGL((given_gather_for<D>(paged, beside)), grid, dim3(kGatherThreads), 0, st, A);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((beside ? given_merge_kernel<D, true, true> : given_merge_kernel<D, true, false>), dim3(p.n_q_heads, pl.vbatch), dim3(D), 0, st,
                     A.part, A.head_rec, A.first_slot + A.splits, p.n_q_heads, out_o, out_lse, pl.group_major, p.n_kv_heads, A.first_slot, A.part_slots);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_sparse_score(const Plan& pl, const void* q, const void* k, const void* v,
                               const int32_t* block_table, const void* rcache, void* ws, const int32_t* out_idx,
                               hipStream_t st) {
  if (pl.p.head_dim == 128) return launch_given_d<128>(pl, 0, q, k, v, block_table, rcache, ws, out_idx, nullptr, nullptr, st);
  if (pl.p.head_dim == 64) return launch_given_d<64>(pl, 0, q, k, v, block_table, rcache, ws, out_idx, nullptr, nullptr, st);
  return hipErrorInvalidValue;
}

hipError_t launch_given_merge(const Plan& pl, void* ws, int splits, float* out_o, float* out_lse, hipStream_t st) {
  const vatt_params& p = pl.p;
  const float* part = reinterpret_cast<const float*>(static_cast<char*>(ws) + pl.off_gather_part);
  const HeadRec* rec = reinterpret_cast<const HeadRec*>(static_cast<char*>(ws) + pl.off_head_rec);
  if (p.head_dim == 128)
    hipLaunchKernelGGL((given_merge_kernel<128, false, false>), dim3(p.n_q_heads, pl.vbatch), dim3(128), 0, st, part, rec, splits,
                       p.n_q_heads, out_o, out_lse, pl.group_major, p.n_kv_heads, 0, splits);
  else if (p.head_dim == 64)
    hipLaunchKernelGGL((given_merge_kernel<64, false, false>), dim3(p.n_q_heads, pl.vbatch), dim3(64), 0, st, part, rec, splits,
                       p.n_q_heads, out_o, out_lse, pl.group_major, p.n_kv_heads, 0, splits);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_given_gather(const Plan& pl, const void* q, const void* k, const void* v,
                               const int32_t* block_table, void* ws, const int32_t* out_idx, float* out_o,
                               float* out_lse, hipStream_t st) {
  if (pl.p.head_dim == 128) return launch_given_d<128>(pl, 1, q, k, v, block_table, nullptr, ws, out_idx, out_o, out_lse, st);
  if (pl.p.head_dim == 64) return launch_given_d<64>(pl, 1, q, k, v, block_table, nullptr, ws, out_idx, out_o, out_lse, st);
  return hipErrorInvalidValue;
}

}  // namespace vatt
