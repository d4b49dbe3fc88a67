// Score pass of a multi-query step (q_len > 1): the q_len newest tokens of every sequence are queries (the question
// tokens of the evaluation set-up in which only the context is processed densely), and every K row is read
// from HBM once for all of them and for all query heads of the GQA group.
//
// With Q query tokens and G heads per KV head, a K tile meets Q * G query vectors: a dense contraction
// [keys x d] . [d x (Q G)], which goes to the matrix cores.  The MFMA v_mfma_f32_16x16x32_bf16 multiplies a 16 x 32
// slice of K (A operand: lane l holds row l % 16, eight consecutive columns starting at 8 (l / 16)) with a 32 x 16 slice
// of the transposed queries (B operand: lane l holds query l % 16, the same eight columns) and accumulates 16 x 16
// scores in fp32 (lane l: keys 4 (l / 16) .. + 3 of query l % 16); d / 32 instructions cover a row.  Products of bf16
// values are exact in fp32, as in the single-query kernel.
//
// Query token t of a sequence of n tokens sees n - (Q - 1 - t) of them; later keys do not enter the 8-key maxima of its
// score row (they count as -inf), which is all the causal mask needs: the selection kernel never looks beyond a row's
// own length.
//
// A wave takes 64 keys at a time and works alone (no workgroup barrier): it requests its K rows, turns them into A
// operands through an LDS tile of its own, and takes the query vectors 16 at a time (16 NQT held in registers; more go
// in rounds) with the K fragments staying in registers.  The 16 x 64 scores of a group pass through the same LDS memory
// so that a wave instruction stores four whole 256-byte pieces of rows, the largest of every 8 keys beside them.  The LDS
// executes the instructions of one wave in order, so a wave's own writes and reads need no barrier.
//
// What bounds it: HBM while there are few vectors; the score rows (4 bytes per key and vector against 256 / (Q G) of K)
// take over as Q grows.  Measured, alone, before (a row of scores per store instruction, its place computed for each)
// and after: 1 x 32K tokens with 2 / 4 / 8 / 16 / 32 query tokens 15.5 / 19.1 / 29 / 52 / 90 -> 14.4 / 16.3 / 20.7 / 28.2 /
// 45.8 us, 16 x 32K with 4 225 -> 216 us, 4 x 128K with 2 211 -> 195 us, 2 x 4K with 10 and groups of 8 21.9 -> 10.3 us.
// Plain stores: 16 x 32K with 4 253 us.
#include <algorithm>
#include <cstring>

#include "vatt_score.h"

namespace vatt {
namespace {

constexpr int kChunkKeys = 64;  // keys a wave takes at a time

struct ChunkArgs {
  const uint16_t* q;
  const uint16_t* k;
  KVLayout L;
  const int32_t* seq_lens;
  float* scores;
  float* sub_max;
  int n_sub, n_pad, n_max, Hq;
  int Q, gshift;  // query tokens; log2 of the group size
  int steps;      // times kChunkKeys keys per wave
  ScoreGrid grid;
  float sm_scale;
};

template <int D, bool PAGED, int NQT>
__global__ __launch_bounds__(64 * kScoreWaves, 2) void score_chunk_kernel(ChunkArgs A) {
  constexpr int S = D / 32, LPR = D / 8, RPI = kWave / LPR, KL = 32 / RPI;
  constexpr int LD = kChunkKeys + 4;  // LDS row stride of the scores: 16-byte aligned, rows 4 banks apart
  static_assert(kSubTile == 8, "two lanes of four keys per sub-tile");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i16 = lane & 15, g4 = lane >> 4, lrow = lane / LPR, lchunk = lane % LPR;
  const int b = blockIdx.z;
  int kvh, chunk;
  score_place(A.grid, (int)blockIdx.y, kvh, chunk);
  const int Q = A.Q, QG = Q << A.gshift;
  const int n = min(max(A.seq_lens[b], 1), A.n_max);
  const int lo = (chunk * A.steps * kScoreWaves + wave) * kChunkKeys;
  const int hi = min(n, (chunk + 1) * A.steps * kScoreWaves * kChunkKeys);
  if (lo >= hi) return;
  union Lds {
    uint4 k[32 * (LPR + 1)];
    float s[16 * LD];
  };
  __shared__ Lds lds_all[kScoreWaves];
  Lds& lds = lds_all[wave];
  uint4 bq[NQT][S];
  // score row of query vector c = (query token c >> gshift, head c mod G of the group)
  auto row_of = [&](int c) { return ((int64_t)b * Q + (c >> A.gshift)) * A.Hq + ((int64_t)kvh << A.gshift) + (c & ((1 << A.gshift) - 1)); };
  auto load_queries = [&](int c0) {
#pragma unroll
    for (int nt = 0; nt < NQT; ++nt) {
      const uint16_t* src = A.q + row_of(min(c0 + nt * 16 + i16, QG - 1)) * D + g4 * 8;
#pragma unroll
      for (int s = 0; s < S; ++s) bq[nt][s] = *reinterpret_cast<const uint4*>(src + s * 32);
    }
  };
  uint4 kr[2][KL];
  auto load_k = [&](int i0) {
    int tab[2][KL];
    auto key = [&](int h, int u) { return min(i0 + 32 * h + u * RPI + lrow, hi - 1); };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int u = 0; u < KL; ++u) tab[h][u] = kv_block<PAGED>(A.L, b, key(h, u));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int u = 0; u < KL; ++u) kr[h][u] = load_stream_16(score_k_at<D, PAGED>(A.k, A.L, b, kvh, key(h, u), tab[h][u], lchunk * 8));
    }
  };
  constexpr int STEP = kScoreWaves * kChunkKeys;
  load_k(lo);
  load_queries(0);
  for (int i0 = lo; i0 < hi; i0 += STEP) {
    uint4 ka[4][S];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int u = 0; u < KL; ++u) lds.k[(u * RPI + lrow) * (LPR + 1) + lchunk] = kr[h][u];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int s = 0; s < S; ++s) ka[2 * h + t][s] = lds.k[(t * 16 + i16) * (LPR + 1) + s * 4 + g4];
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (i0 + STEP < hi) load_k(i0 + STEP);
    const bool edge = i0 + kChunkKeys > n - Q + 1;
    for (int c0 = 0; c0 < QG; c0 += 16 * NQT) {
      if (QG > 16 * NQT) load_queries(c0);
#pragma unroll
      for (int nt = 0; nt < NQT; ++nt) {
        if (c0 + nt * 16 >= QG) break;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < S; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[t][s]),
                                                          __builtin_bit_cast(bf16x8_t, bq[nt][s]), acc, 0, 0, 0);
          *reinterpret_cast<float4*>(&lds.s[i16 * LD + t * 16 + 4 * g4]) =
              make_float4(acc[0] * A.sm_scale + 0.0f, acc[1] * A.sm_scale + 0.0f, acc[2] * A.sm_scale + 0.0f, acc[3] * A.sm_scale + 0.0f);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = c0 + nt * 16 + 4 * j + g4;
          const float4 o = *reinterpret_cast<const float4*>(&lds.s[(4 * j + g4) * LD + 4 * i16]);
          const int64_t row = row_of(min(c, QG - 1));
          const int i = i0 + 4 * i16;
          if (c < QG) {
            f32x4_t* dst = reinterpret_cast<f32x4_t*>(A.scores + row * A.n_pad + i);
            const f32x4_t oo = {o.x, o.y, o.z, o.w};
            __builtin_nontemporal_store(oo, dst);
          }
          float m = edge ? max4_seen(o, max(n - (Q - 1 - (c >> A.gshift)), 1), i) : fmaxf(fmaxf(o.x, o.y), fmaxf(o.z, o.w));
          m = fmaxf(m, dpp_f32<0xB1>(m));
          if (c < QG && (lane & 1) == 0) A.sub_max[row * A.n_sub + i / kSubTile] = m;
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

template <int D, bool PAGED>
hipError_t launch_p(const Plan& pl, ChunkArgs& A, hipStream_t st) {
  const vatt_params& p = pl.p;
  // Small caches (up to 256 MB of K) go KV head by KV head with two steps per wave, where that leaves at least two
  // workgroups per CU: 1 x 32K tokens with 4 / 16 query tokens 17.3 / 33.6 -> 16.3 / 28.2 us.  Large ones tile by tile, one
  // step per wave (16 x 32K with 4 216 us, KV head by KV head 224; 4 x 128K with 2 195 and 226).
  const size_t k_bytes = (size_t)p.batch * p.n_kv_heads * p.n_max * D * 2;
  const bool small = k_bytes <= (size_t)256 * 1024 * 1024;
  auto chunks = [&](int steps) { return (p.n_max + steps * kScoreWaves * kChunkKeys - 1) / (steps * kScoreWaves * kChunkKeys); };
  A.steps = small && (int64_t)chunks(2) * p.n_kv_heads * p.batch >= 2 * pl.num_cus ? 2 : 1;
  const dim3 grid = score_grid(A.grid, small && pl.group_major ? kScoreOrderKvHead : kScoreOrderTile, chunks(A.steps),
                               (size_t)A.steps * kScoreWaves * kChunkKeys * D * 2, p.n_kv_heads, p.batch);
  const int groups = (pl.q_len * pl.group + 15) / 16;  // (more than 64 query vectors go in rounds of 32: measured best)
  if (groups == 1) hipLaunchKernelGGL((score_chunk_kernel<D, PAGED, 1>), grid, dim3(64 * kScoreWaves), 0, st, A);
  else if (groups == 2 || groups > 4) hipLaunchKernelGGL((score_chunk_kernel<D, PAGED, 2>), grid, dim3(64 * kScoreWaves), 0, st, A);
  else hipLaunchKernelGGL((score_chunk_kernel<D, PAGED, 4>), grid, dim3(64 * kScoreWaves), 0, st, A);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_chunk(const Plan& pl, const void* q, const void* k, const int32_t* block_table,
                              const int32_t* seq_lens, void* ws, hipStream_t st) {
  const vatt_params& p = pl.p;
  char* w = static_cast<char*>(ws);
  ChunkArgs A;
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
  A.Q = pl.q_len;
  while ((1 << A.gshift) < pl.group) ++A.gshift;
  A.sm_scale = pl.sm_scale;
  const bool paged = p.kv_layout == VATT_LAYOUT_PAGED;
  if (p.head_dim == 128) return paged ? launch_p<128, true>(pl, A, st) : launch_p<128, false>(pl, A, st);
  if (p.head_dim == 64) return paged ? launch_p<64, true>(pl, A, st) : launch_p<64, false>(pl, A, st);
  return hipErrorInvalidValue;
}

}  // namespace vatt
