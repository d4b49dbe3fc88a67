// What the two score kernels share (vatt_score.hip: one query token; vatt_score_chunk.hip: several): which piece of
// a score row a workgroup owns, and the addresses of the K rows that a wave reads.
#pragma once
#include "vatt_internal.h"

namespace vatt {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kScoreWaves = 4;  // waves per workgroup; they do not interact

// Launch grid of a score pass over `chunks` pieces of every (KV head, sequence), and back.  Workgroups go to the
// chip's eight XCDs round-robin in launch order, so the order decides which XCD reads which piece of K and writes which
// piece of a score row:
//   tile by tile, grid = (chunks, KV heads, sequences): the XCDs take turns along every row;
//   KV-head-major, grid = (KV heads, chunks, sequences): with a multiple of 8 KV heads every XCD streams the rows of
//     its own KV heads front to back and writes whole score rows;
//   blocks: as tile by tile, but the XCDs take turns in blocks of 256 KiB of K; which XCD starts a row rotates with
//     the KV head and the sequence, so that the first blocks, all that a short sequence has, do not land on one XCD.
struct ScoreGrid {
  int order;
  int block;  // blocks order: chunks per block
};
inline dim3 score_grid(ScoreGrid& g, int order, int chunks, size_t chunk_bytes, int n_kv_heads, int batch) {
  g.order = order;
  g.block = (int)(chunk_bytes < 256 * 1024 ? 256 * 1024 / chunk_bytes : 1);
  if (order == kScoreOrderKvHead) return dim3(n_kv_heads, chunks, batch);
  if (order == kScoreOrderBlocks) chunks = (chunks + 8 * g.block - 1) / (8 * g.block) * (8 * g.block);  // whole groups of eight blocks
  return dim3(chunks, n_kv_heads, batch);
}
// (row: blockIdx.y, less the rows of the grid that do something else)
__device__ __forceinline__ void score_place(const ScoreGrid& g, int row, int& kvh, int& chunk) {
  const int x = (int)blockIdx.x;
  if (g.order == kScoreOrderKvHead) {
    kvh = x;
    chunk = row;
  } else {
    kvh = row;
    chunk = g.order == kScoreOrderBlocks ? ((x / 8 / g.block) * 8 + (x + row + (int)blockIdx.z) % 8) * g.block + (x / 8) % g.block : x;
  }
}

// Column c of K row i (contiguous cache: a uniform address and 32-bit offsets, which take fewest registers; at most
// 170752 tokens).
template <int D, bool PAGED>
__device__ __forceinline__ const uint16_t* score_k_at(const uint16_t* k, const KVLayout& L, int b, int kvh, int i, int blk, int c) {
  if constexpr (PAGED) return k + kv_row_offset_in<true>(L, b, kvh, i, blk) + c;
  else return k + kv_row_offset<false>(L, b, kvh, 0) + (uint32_t)(i * D + c);
}

// Largest of four scores of keys i .. i + 3, of which those at `seen` and beyond do not count.
__device__ __forceinline__ float max4_seen(float4 o, int seen, int i) {
  const int left = seen - i;
  o.x = left > 0 ? o.x : -INFINITY;
  o.y = left > 1 ? o.y : -INFINITY;
  o.z = left > 2 ? o.z : -INFINITY;
  o.w = left > 3 ? o.w : -INFINITY;
  return fmaxf(fmaxf(o.x, o.y), fmaxf(o.z, o.w));
}

}  // namespace
}  // namespace vatt
