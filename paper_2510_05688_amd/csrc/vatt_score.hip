// Score pass: s_i = sm_scale * <K[i], q_h> for every key and every query head of the GQA group,
// reading each K row from HBM once per group (first step of Algorithm 1 with exact top-k; the
// exponent of Eq. 1).
//
// Work split: a wave takes 16 or 32 consecutive keys, a workgroup of four waves 64 or 128, and does nothing else: many
// short workgroups fill and drain the chip more evenly than few long ones (4 to 16 steps a wave with the next rows
// requested under the current ones: 186 to 205 us for 16 x 32K, against 176).  d/8 adjacent lanes read a K row with one
// 16-byte load each, so a wave instruction covers whole rows as one contiguous KiB, and all rows of a wave are in flight
// together.  Each lane multiplies its 8 columns with those of the G queries (bf16 pair dot products into fp32), the
// partial sums are added across the lanes of the row on the DPP path, and the scores pass through LDS so that they leave
// as lines of 64 to 256 bytes, the largest of every 8 keys beside them.  A wave writes its own piece (the LDS executes
// the instructions of one wave in order: no barrier) except where a group of at most four heads of 64 columns leaves so
// little per wave that the workgroup writes together.
//
// Keys per wave, by measurement (whole call, before -> after, us; before: 64 keys per workgroup, 256 on a paged cache,
// and an exchange of 4 G additions per row):
//   32 on a paged cache, whose block-table reads then come once per 32 rows and beside 7 other waves of them: 8 of
//     0.5K - 7K tokens 56.5 -> 48.2, 32 of 1K - 33K with 16-token pages 327 -> 319 (16 keys: 330), 16 x 32K 284 -> 272;
//   32 for groups of 8, where the arithmetic counts: 8 x 20K 80.6 -> 77 (16 keys: 79);
//   else 16: 16 x 32K 258 -> 251 (32 keys: 260), 1 x 32K 38.3 -> 37.6 (38.6); with 64 columns written by the whole
//     workgroup: 8 x 40K of 16 KV heads 152 (32 keys or each wave for itself: 155).
// What bounds it: K is read at the pace of a kernel that only reads (16 x 32K: 1.07 GB in 176 us, 6.1 TB/s of K, 6.5
// with the scores); the scores, a sixteenth of the bytes at G = 4, cost a further sixth of the time, which is this memory system's
// price for writes among reads.  K loads without the non-temporal hint take 2.5 times as long.
#include <cstring>

#include "vatt_sampler.h"
#include "vatt_score.h"

namespace vatt {
namespace {

// Keys of a wave, and whether the four waves of a workgroup write their scores together (see above).
template <int D, int G, bool PAGED>
constexpr int score_keys() { return G <= 4 && !PAGED ? 16 : 32; }
template <int D, int G, bool PAGED>
constexpr bool score_joint() { return D == 64 && G <= 4 && !PAGED; }

struct ScoreArgs {
  const uint16_t* q;
  const uint16_t* k;
  KVLayout L;
  const int32_t* seq_lens;
  float* scores;
  float* sub_max;
  int n_sub, n_pad, n_max, Hq;
  ScoreGrid grid;
  float sm_scale;
  PreArgs pre;
};

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc,
                                         false);
}

// <K row, q_g> for the G queries of a group, from the 8 columns of each of the LPR adjacent lanes that hold the row;
// lane `sub` < G of them gets head sub's.  A lane's columns are summed first, then lanes ^ 1, ^ 2, quads, halves.  Where
// two lanes hold the partial sums of two heads, each takes one head from both (one addition for the two, with two
// selections), so that four heads cost 11 instructions of exchange instead of 16 and a selection each.
template <int G, int LPR>
__device__ __forceinline__ float group_scores(const uint4& k, const uint32_t (&qw)[G][4], int sub) {
  const bool odd = sub & 1, two = sub & 2;
  float a[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    a[g] = dot2_bf16(k.x, qw[g][0], 0.f);
    a[g] = dot2_bf16(k.y, qw[g][1], a[g]);
    a[g] = dot2_bf16(k.z, qw[g][2], a[g]);
    a[g] = dot2_bf16(k.w, qw[g][3], a[g]);
  }
  float v;
  if constexpr (G == 1) {
    v = a[0] + dpp_f32<0xB1>(a[0]);
    v += dpp_f32<0x4E>(v);
    v += dpp_f32<0x104>(v);
  } else {
    float p[G / 2];
#pragma unroll
    for (int j = 0; j < G / 2; ++j) p[j] = (odd ? a[2 * j + 1] : a[2 * j]) + dpp_f32<0xB1>(odd ? a[2 * j] : a[2 * j + 1]);
    if constexpr (G == 2) {
      v = p[0] + dpp_f32<0x4E>(p[0]);
      v += dpp_f32<0x104>(v);
    } else {
      float r[G / 4];
#pragma unroll
      for (int j = 0; j < G / 4; ++j) r[j] = (two ? p[2 * j + 1] : p[2 * j]) + dpp_f32<0x4E>(two ? p[2 * j] : p[2 * j + 1]);
      v = r[0] + dpp_f32<0x104>(r[0]);  // row_shl:4, right for the even quads
      if constexpr (G == 8) {
        const float w = r[1] + dpp_f32<0x114>(r[1]);  // row_shr:4, right for the odd ones
        v = (sub & 4) ? w : v;
      }
    }
  }
  if constexpr (LPR == 16) v += dpp_f32<0x108>(v);  // row_shl:8, right for the lower half
  return v;
}

template <int D, int G, bool PAGED, bool NT>
__global__ __launch_bounds__(64 * kScoreWaves, 4) void score_kernel(ScoreArgs A) {
  constexpr int LPR = D / 8;
  constexpr int RPI = kWave / LPR;
  constexpr int KEYS = score_keys<D, G, PAGED>();
  constexpr int KL = KEYS / RPI;
  constexpr bool JOINT = score_joint<D, G, PAGED>();
  constexpr int SPAN = JOINT ? kScoreWaves * KEYS : KEYS;  // keys that are written together
  constexpr int LD = SPAN + 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rsub = lane / LPR, sub = lane % LPR;
  // sampler pre-work: the first pre.job_rows rows of the grid (the workgroups that start first) each make the first
  // batch of draws of one (head, stream) and are done
  if (A.pre.job_rows > 0 && (int)blockIdx.y < A.pre.job_rows) {
    extern __shared__ __align__(16) unsigned char pre_smem[];
    const int job = (int)blockIdx.y * (int)gridDim.x + (int)blockIdx.x;
    if (job < 2 * A.Hq) prework_job(A.pre, (int)blockIdx.z, job >> 1, job & 1, pre_smem);
    return;
  }
  const int b = blockIdx.z;
  int kvh, chunk;
  score_place(A.grid, (int)blockIdx.y - A.pre.job_rows, kvh, chunk);
  const int n = min(max(A.seq_lens[b], 1), A.n_max);
  const int lo = (chunk * kScoreWaves + wave) * KEYS;
  if ((JOINT ? chunk * kScoreWaves * KEYS : lo) >= n) return;
  static_assert(kSubTile == 8, "two lanes of four keys per sub-tile");
  constexpr int ROWS = JOINT ? G : kWave * 4 / KEYS;
  __shared__ __align__(16) float s_all[JOINT ? 1 : kScoreWaves][ROWS * LD];
  float* s_tile = s_all[JOINT ? 0 : wave] + (JOINT ? wave * KEYS : 0);

  auto key = [&](int u) { return min(lo + u * RPI + rsub, n - 1); };
  int tab[KL];
#pragma unroll
  for (int u = 0; u < KL; ++u) tab[u] = kv_block<PAGED>(A.L, b, key(u));
  uint4 kr[KL];
#pragma unroll
  for (int u = 0; u < KL; ++u) kr[u] = load_stream_16(score_k_at<D, PAGED>(A.k, A.L, b, kvh, key(u), tab[u], sub * 8));
  const int64_t row0 = (int64_t)b * A.Hq + (int64_t)kvh * G;
  uint32_t qw[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 t = *reinterpret_cast<const uint4*>(A.q + (row0 + g) * D + sub * 8);
    qw[g][0] = t.x; qw[g][1] = t.y; qw[g][2] = t.z; qw[g][3] = t.w;
  }
#pragma unroll
  for (int u = 0; u < KL; ++u) {
    const float v = group_scores<G, LPR>(kr[u], qw, sub);
    // adding +0 folds a possible -0 into +0 so that the bit pattern orders like the value
    if (sub < G) s_tile[sub * LD + u * RPI + rsub] = v * A.sm_scale + 0.0f;
  }
  if constexpr (JOINT) __syncthreads();
  else __builtin_amdgcn_wave_barrier();
  const int t = JOINT ? (int)threadIdx.x : lane;
  const int orow = t / (SPAN / 4), okey = (JOINT ? -wave * KEYS : 0) + (t % (SPAN / 4)) * 4;  // row and keys this lane stores
  if (JOINT && orow >= G) return;
  const float4 o = *reinterpret_cast<const float4*>(&s_tile[orow * LD + okey]);
  float m = lo + okey + 4 > n ? max4_seen(o, n, lo + okey) : fmaxf(fmaxf(o.x, o.y), fmaxf(o.z, o.w));
  m = fmaxf(m, dpp_f32<0xB1>(m));
  if (orow < G) {
    f32x4_t* dst = reinterpret_cast<f32x4_t*>(A.scores + (row0 + orow) * A.n_pad + lo + okey);
    const f32x4_t oo = {o.x, o.y, o.z, o.w};
    if (NT) __builtin_nontemporal_store(oo, dst); else *dst = oo;
    if ((lane & 1) == 0) A.sub_max[(row0 + orow) * A.n_sub + (lo + okey) / kSubTile] = m;
  }
}

template <int D, int G, bool PAGED>
hipError_t launch_g(const Plan& pl, ScoreArgs& A, hipStream_t st) {
  const vatt_params& p = pl.p;
  constexpr int keys = kScoreWaves * score_keys<D, G, PAGED>();
  // Non-temporal stores for score rows that the selection kernel would not find in the last-level cache anyway, where its
  // heads are enough to hide the time to memory: it then takes 5 us longer and the score pass 12 us less.  Whole call, plain ->
  // non-temporal, us: 16 x 32K 267.6 -> 258.7, 8 x 64K 276 -> 265, 8 x 32K 146.6 -> 143.6, 16 x 16K 160.3 -> 157.5, 32 x 8K 198.6 ->
  // 195.8, 64 x 4K 269.7 -> 265.9, 4 x 128K 255.2 -> 252.7, 32 of 1K - 33K on pages 315.5 -> 310.8, and equal at 4 x 64K (153.1,
  // 156.3, runs 3 apart); below the limits 2 x 128K 208 -> 210, 8 x 16K 86.1 -> 86.0.  (By the counters the pass then writes 84.3 MB
  // instead of 75.5 at 16 x 32K.)
  const bool nt = score_bytes(pl) >= kScoreBytesLarge && p.batch * p.n_q_heads >= 128;
  dim3 grid = score_grid(A.grid, pl.score_order, (p.n_max + keys - 1) / keys, (size_t)keys * D * 2, p.n_kv_heads, p.batch);
  size_t lds = 0;
  if (A.pre.pre_tok) {
    A.pre.job_rows = (2 * p.n_q_heads + (int)grid.x - 1) / (int)grid.x;
    grid.y += A.pre.job_rows;
    lds = prework_lds_bytes(p.n_max);
  }
  if (nt) hipLaunchKernelGGL((score_kernel<D, G, PAGED, true>), grid, dim3(64 * kScoreWaves), lds, st, A);
  else hipLaunchKernelGGL((score_kernel<D, G, PAGED, false>), grid, dim3(64 * kScoreWaves), lds, st, A);
  return hipGetLastError();
}

template <int D, bool PAGED>
hipError_t launch_p(const Plan& pl, ScoreArgs& A, hipStream_t st) {
  switch (pl.group) {
    case 1: return launch_g<D, 1, PAGED>(pl, A, st);
    case 2: return launch_g<D, 2, PAGED>(pl, A, st);
    case 4: return launch_g<D, 4, PAGED>(pl, A, st);
    case 8: return launch_g<D, 8, PAGED>(pl, A, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_score(const Plan& pl, const void* q, const void* k, const int32_t* block_table,
                        const int32_t* seq_lens, const uint64_t* seq_seeds, void* ws, hipStream_t st) {
  const vatt_params& p = pl.p;
  char* w = static_cast<char*>(ws);
  ScoreArgs A;
  memset(&A, 0, sizeof(A));
  A.q = static_cast<const uint16_t*>(q);
  A.k = static_cast<const uint16_t*>(k);
  A.L = pl.kv_k;
  A.L.block_table = block_table;
  A.seq_lens = seq_lens;
  A.scores = reinterpret_cast<float*>(w + pl.off_scores);
  A.sub_max = reinterpret_cast<float*>(w + pl.off_sub_max);
  A.n_sub = pl.n_sub;
  A.n_pad = pl.n_pad;
  A.n_max = p.n_max;
  A.Hq = p.n_q_heads;
  A.sm_scale = pl.sm_scale;
  if (score_prework(pl) && seq_seeds) {
    A.pre.seq_lens = seq_lens;
    A.pre.seq_seeds = seq_seeds;
    A.pre.pre_tok = reinterpret_cast<uint4*>(w + pl.off_pre_tok);
    A.pre.pre_flags = reinterpret_cast<uint32_t*>(w + pl.off_pre_flags);
    A.pre.sp = pl.sel;
    A.pre.n_max = p.n_max;
    A.pre.Hq = p.n_q_heads;
    A.pre.small_batches = pl.sampler_small_batches;
    A.pre.draw_cap = pl.sampler_draw_cap;
  }
  const bool paged = p.kv_layout == VATT_LAYOUT_PAGED;
  if (p.head_dim == 128) return paged ? launch_p<128, true>(pl, A, st) : launch_p<128, false>(pl, A, st);
  if (p.head_dim == 64) return paged ? launch_p<64, true>(pl, A, st) : launch_p<64, false>(pl, A, st);
  return hipErrorInvalidValue;
}

}  // namespace vatt
