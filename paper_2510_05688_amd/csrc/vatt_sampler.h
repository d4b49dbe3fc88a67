// The sampler of Algorithm 1 and Algorithm 2 as device code shared by the selection kernels and by the score
// kernel (which can make the first batch of draws of every head while it streams K): sequential uniform draws
// from the middle region (Philox4x32-10 words, unbiased multiply-and-reject mapping), skipping top-k members and
// tokens drawn before; the first c accepted tokens are the sample.  The draw sequence is processed in batches:
// all draws of a batch are generated at once, repeated tokens are resolved to their earliest draw, and a
// prefix count in draw order finds where the sample is complete; the result equals the sequential procedure
// bit for bit.
#pragma once

#include "vatt_dev.h"

namespace vatt {

constexpr uint32_t kInv32 = 0xffffffffu;
// Mail slots in which the draws of repeated tokens find their earliest one (a power of two; the slot number and 8
// more bits make a token, see kCapacityMax).
constexpr uint32_t kMailSlots = 2048;
constexpr int kMailTokens = 256;  // tokens that 8 bits tell apart in a slot
// 32-bit words of a bitmap over n_max tokens: whole groups of four, which one store clears.
__host__ __device__ constexpr int bitmap_words(int n_max) { return ((n_max + 127) >> 7) << 2; }

// ---------------------------------------------------------------------------
// Workgroup-wide exclusive scan of one uint32 per thread (DPP inside a wave, LDS across waves).
// ---------------------------------------------------------------------------
template <int NT>
struct BlockScanSmem {
  uint32_t wave_total[NT / kWave];
};
// Returns the exclusive prefix of v; *total gets the workgroup sum.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total, BlockScanSmem<NT>& sm) {
  constexpr int SW = NT / kWave;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan_u32(v);
  __syncthreads();  // protects wave_total against a previous use
  if (lane == kWave - 1) sm.wave_total[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SW; ++w) {
    const uint32_t t = sm.wave_total[w];
    base += (w < wave) ? t : 0u;
    tot += t;
  }
  *total = tot;
  return base + incl - v;
}

// The same with shared memory that nothing else uses in this launch: one barrier.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan_once(uint32_t v, uint32_t* total, BlockScanSmem<NT>& sm) {
  constexpr int SW = NT / kWave;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan_u32(v);
  if (lane == kWave - 1) sm.wave_total[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SW; ++w) {
    const uint32_t t = sm.wave_total[w];
    base += (w < wave) ? t : 0u;
    tot += t;
  }
  *total = tot;
  return base + incl - v;
}

// Two of them at once: a and b become their exclusive prefixes, *total_b gets the workgroup sum of b.
template <int NT>
__device__ __forceinline__ void block_exclusive_scan_two_once(uint32_t& a, uint32_t& b, uint32_t* total_b, BlockScanSmem<NT>& sa,
                                                              BlockScanSmem<NT>& sb) {
  constexpr int SW = NT / kWave;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl_a = wave_inclusive_scan_u32(a), incl_b = wave_inclusive_scan_u32(b);
  if (lane == kWave - 1) {
    sa.wave_total[wave] = incl_a;
    sb.wave_total[wave] = incl_b;
  }
  __syncthreads();
  uint32_t base_a = 0, base_b = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SW; ++w) {
    const uint32_t ta = sa.wave_total[w], tb = sb.wave_total[w];
    base_a += (w < wave) ? ta : 0u;
    base_b += (w < wave) ? tb : 0u;
    tot += tb;
  }
  *total_b = tot;
  a = base_a + incl_a - a;
  b = base_b + incl_b - b;
}

// Number of the set bits of a wave's mask that belong to lower lanes.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Where an accepted token goes: into the index list in global memory (dst, for the workgroup that writes the
// outputs) and, when a workgroup gathers its own share of the list (fused gather), every 2^shift-th entry into
// an LDS list.
struct Emit {
  int32_t* dst;
  uint32_t dst_cap;
  uint32_t* lds;      // nullptr: no LDS list
  uint32_t lds_cap;
  uint32_t shift, split;
  bool global;
  float* sc_dst;      // nullptr, or where the scores of the listed tokens go when the batch has them at hand
};
__device__ __forceinline__ void emit_tok(const Emit& E, uint32_t p, int32_t tok) {
  if (E.global && p < E.dst_cap) E.dst[p] = tok;
  if (E.lds && (p & ((1u << E.shift) - 1u)) == E.split && (p >> E.shift) < E.lds_cap) E.lds[p >> E.shift] = (uint32_t)tok;
}
__device__ __forceinline__ Emit emit_to(int32_t* dst, uint32_t dst_cap) {
  Emit E;
  E.dst = dst;
  E.dst_cap = dst_cap;
  E.lds = nullptr;
  E.lds_cap = 0;
  E.shift = 0;
  E.split = 0;
  E.global = true;
  E.sc_dst = nullptr;
  return E;
}

constexpr int kSmallBatchBlocks = 64;  // Philox blocks of a small batch (256 draws)

// flag bits of out_counts[7]
constexpr int kFlagBaseComplement = 1, kFlagDynComplement = 2, kFlagBaseBatches = 4, kFlagDynBatches = 8,
              kFlagDrawCap = 16, kFlagTopkGeneral = 32, kFlagBaseFromCache = 64;

// One batch of the draw sequence as a thread sees it: the four draws of one Philox block.
struct DrawBatch {
  uint32_t tok[4];  // proposed tokens
  float sc[4];      // their scores, when loaded ahead
  uint32_t ok;      // bit e: the draw counts (inside the batch and the draw cap, word not rejected, token not
                    // drawn in an earlier batch)
  uint32_t first;   // bit e: ok and no earlier draw of the batch proposes the same token
  int blocks;       // Philox blocks in the batch
  bool have_sc;
};

// Device functions of the per-head kernel for a workgroup of NT threads.
template <int NT>
struct HeadOps {
  static constexpr int SW = NT / kWave;

  struct HeadSmem {
    BlockScanSmem<NT> scan;
    double red[3][SW];
    uint32_t again[2];
    uint32_t last_block;  // Philox block that completed a sample
    BlockScanSmem<NT> scan_once[4];  // for scans that run once in a launch and need no barrier before them
  };

  // Workgroup sums of up to three doubles at once; every thread gets all of them.  (The sums of the waves are added
  // by groups of 16 lanes of every wave, one group per sum, instead of by every thread.)
  template <int N>
  static __device__ __forceinline__ void block_sum(double (&v)[N], HeadSmem& sm) {
    __syncthreads();
    block_sum_post(v, sm);
    __syncthreads();
    block_sum_get(v, sm);
  }
  // Its two halves, for callers that have a barrier between them anyway.
  template <int N>
  static __device__ __forceinline__ void block_sum_post(double (&v)[N], HeadSmem& sm) {
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = wave_sum(v[j]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int j = 0; j < N; ++j) sm.red[j][threadIdx.x >> 6] = v[j];
    }
  }
  template <int N>
  static __device__ __forceinline__ void block_sum_get(double (&v)[N], const HeadSmem& sm) {
    static_assert(N <= 4 && SW <= 16, "a row of 16 lanes per sum");
    const int row = (int)(threadIdx.x & 63) >> 4, w = (int)(threadIdx.x & 15);
    double t = sm.red[min(row, N - 1)][min(w, SW - 1)];
    t = w < SW ? t : 0.0;
    t += dpp_f64<0xB1>(t);
    t += dpp_f64<0x4E>(t);
    t += dpp_f64<0x141>(t);
    t += dpp_f64<0x140>(t);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = readlane_f64(t, 16 * j);
  }
  // Token read back from an index list, forced into [0, n): a list entry can never address outside the row.
  static __device__ __forceinline__ int list_tok(const int32_t* idx, int64_t pos, int n) {
    return min(max(idx[pos], 0), n - 1);
  }

  static __device__ __forceinline__ void mark_bit(uint32_t* bm, uint32_t i) { atomicOr(&bm[i >> 5], 1u << (i & 31)); }
  static __device__ __forceinline__ bool test_bit(const uint32_t* bm, uint32_t i) { return (bm[i >> 5] >> (i & 31)) & 1u; }
  // Bit e of the result: the bitmap bit of tok[e].  All four words are read before any is used (a test per token
  // behind a condition compiles to four LDS round trips one after the other); every token has to be a valid one.
  static __device__ __forceinline__ uint32_t test_bits4(const uint32_t* bm, const uint32_t (&tok)[4]) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = bm[tok[e] >> 5];
    uint32_t r = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) r |= ((w[e] >> (tok[e] & 31)) & 1u) << e;
    return r;
  }

  // Exclusive prefix of the set-bit counts of bm[0, words) into wpre; returns the number of set bits.
  // once: scan memory that nothing else uses in this launch (saves a barrier), or nullptr.
  static __device__ uint32_t word_prefix(const uint32_t* bm, int words, uint32_t* wpre, HeadSmem& sm,
                                         BlockScanSmem<NT>* once = nullptr) {
    const int wpt = (words + NT - 1) / NT;
    const int w0 = threadIdx.x * wpt;
    uint32_t cnt = 0;
    for (int w = w0; w < min(w0 + wpt, words); ++w) cnt += __popc(bm[w]);
    uint32_t total;
    uint32_t pos = once ? block_exclusive_scan_once<NT>(cnt, &total, *once) : block_exclusive_scan<NT>(cnt, &total, sm.scan);
    for (int w = w0; w < min(w0 + wpt, words); ++w) {
      wpre[w] = pos;
      pos += __popc(bm[w]);
    }
    __syncthreads();
    return total;
  }

  // Bits of word w that lie in the middle region [mid_lo, mid_hi).
  static __device__ __forceinline__ uint32_t mid_mask(const HeadSizes& hs, int w) {
    const int i0 = w << 5;
    if (i0 + 31 < hs.mid_lo || i0 >= hs.mid_hi) return 0u;
    const int a = max(hs.mid_lo - i0, 0), bnd = min(hs.mid_hi - i0, 32);
    return (bnd >= 32 ? 0xffffffffu : ((1u << bnd) - 1u)) & ~((1u << a) - 1u);
  }

  // What one sample needs to know.
  struct Sampler {
    uint32_t* taken;      // tokens proposed so far (bitmap, LDS)
    uint32_t* scratch;    // all-zero bitmap between uses (LDS)
    uint32_t* mail;       // kMailSlots slots, free between batches (LDS)
    const uint32_t* bm_f; // top-k members (bitmap, LDS)
    uint32_t* wpre;       // word prefixes (LDS)
    const float* row;     // the head's scores
    uint64_t seed;
    uint32_t stream, head, query;
    uint32_t L, thr;      // middle-region length and 2^32 mod L
    uint32_t cap;         // draws allowed
    float m;
    unsigned long long* dbg;
  };

  // Generate the draws of Philox blocks [blk0, blk0 + blocks) of the stream and find, for every token that is
  // proposed more than once in the batch, its earliest draw.
  //
  // Every draw that counts sets its token's bit in `taken`; a draw that finds the bit already set knows that
  // the token is repeated and says so in `scratch`.  The draws of repeated tokens then post (draw number, upper
  // token bits) with an atomic minimum into the mail slot of their token (its lower bits); the smallest draw
  // number of a token wins its slot.  Two repeated tokens that share a slot take turns (one more round per token).
  // (Slots by token, not by bitmap word: 1024 draws from a thousand tokens repeat a dozen tokens in every word, and
  // as many rounds took 22 K of the 71 K clocks of the selection kernel on a 1K-token row, more on shorter ones.
  // Rows of up to kMailSlots tokens now need one round.)
  //
  // lt: the Philox block (relative to blk0) this thread generates, normally its thread index.  Two streams can
  // share one call, each thread working for one of them (its own S, with bitmaps, scratch and mail of that
  // stream, and lt counted inside the stream's group of threads): the barriers are common, the rest is per
  // thread.
  static __device__ __forceinline__ void make_batch(DrawBatch& B, const Sampler& S, const HeadSizes& hs, uint32_t blk0, int blocks,
                                    bool check_prev, bool load_scores, HeadSmem& sm, int lt) {
    const int tid = lt;
    B.blocks = blocks;
    B.ok = 0;
    B.first = 0;
    B.have_sc = load_scores;
    VATT_STAMP(S.dbg, 0);
    if (tid >= 0 && tid < blocks) {
      const Philox4 ph = philox4x32_10(blk0 + (uint32_t)tid, S.stream, S.head, S.query, (uint32_t)S.seed,
                                       (uint32_t)(S.seed >> 32));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t j = ((blk0 + (uint32_t)tid) << 2) + (uint32_t)e;
        const uint64_t x = (uint64_t)ph.v[e] * (uint64_t)S.L;
        const uint32_t t = (uint32_t)hs.mid_lo + (uint32_t)(x >> 32);
        bool v = j < S.cap && (uint32_t)x >= S.thr;
        if (check_prev) v = v && !test_bit(S.taken, t);
        B.tok[e] = t;
        B.ok |= (v ? 1u : 0u) << e;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) B.tok[e] = (uint32_t)hs.mid_lo;
    }
    if (load_scores) {
#pragma unroll
      for (int e = 0; e < 4; ++e) B.sc[e] = S.row[B.tok[e]];
    }
    VATT_STAMP(S.dbg, 1);
    if (check_prev) __syncthreads();  // every test of `taken` comes before the marks of this batch
    // (the four marks go out together: a void draw ORs in nothing)
    uint32_t lose = 0, old[4] = {0u, 0u, 0u, 0u};
    if (B.ok) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        old[e] = atomicOr(&S.taken[B.tok[e] >> 5], ((B.ok >> e) & 1u) << (B.tok[e] & 31));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t bit = ((B.ok >> e) & 1u) << (B.tok[e] & 31);
      if (old[e] & bit) {
        lose |= 1u << e;
        atomicOr(&S.scratch[B.tok[e] >> 5], bit);
      }
    }
    __syncthreads();
    VATT_STAMP(S.dbg, 2);
    // draws whose token is proposed more than once in this batch
    uint32_t unresolved = B.ok & test_bits4(S.scratch, B.tok);
    uint32_t later = 0;
    // (a round settles a token of every slot in question, and no more than kMailTokens share one)
    for (int round = 0; round < kMailTokens; ++round) {
      // (the slots in question are cleared first; the flag alternates, so that it can be cleared here as well)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((unresolved >> e) & 1u) S.mail[B.tok[e] % kMailSlots] = kInv32;
      if (threadIdx.x == 0) sm.again[round & 1] = 0;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((unresolved >> e) & 1u)
          atomicMin(&S.mail[B.tok[e] % kMailSlots], ((uint32_t)(tid * 4 + e) << 8) | (B.tok[e] / kMailSlots));
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if ((unresolved >> e) & 1u) {
          const uint32_t v = S.mail[B.tok[e] % kMailSlots];
          if ((v & 255u) == B.tok[e] / kMailSlots) {
            if ((v >> 8) != (uint32_t)(tid * 4 + e)) later |= 1u << e;
            unresolved &= ~(1u << e);
          }
        }
      }
      if (unresolved) sm.again[round & 1] = 1;
      __syncthreads();
      if (sm.again[round & 1] == 0) break;
    }
    B.first = B.ok & ~later;
    VATT_STAMP(S.dbg, 3);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((lose >> e) & 1u) atomicAnd(&S.scratch[B.tok[e] >> 5], ~(1u << (B.tok[e] & 31)));
    __syncthreads();
    VATT_STAMP(S.dbg, 4);
  }

  // Philox blocks of a batch when `remaining` accepted draws are asked for.
  static __device__ __forceinline__ int first_blocks(int small_batches, uint32_t remaining) {
    return (small_batches || remaining <= 128u) ? kSmallBatchBlocks : (remaining > 1024u ? min(NT, 1024) : min(NT, 256));
  }

  // Draw a sample of c residual tokens for the stream described by S.  `taken` must be all zero on entry
  // unless `spec` carries the first batch (have_spec; made from block 0 with make_batch), `scratch` all zero.
  // Writes the token list to dst (acceptance order, or ascending when the sample is a complement) and, when
  // sum_w is given, adds exp(s_i - m) and its square over the sample to this thread's partial sums.
  // have, blk: the first `have` tokens, from the Philox blocks before blk, are listed already (no complement).
  // Returns flag bits: 1 complement regime, 2 more than one batch, 4 draw cap reached.  by_rule: bit 2 says whether the sample
  // needs more than a first batch of rule_blocks (0: first_blocks()), whatever batches it was made from.
  static __device__ __forceinline__ int draw_sample(const Sampler& S, const HeadSizes& hs, uint32_t c, const DrawBatch& spec, bool have_spec,
                                    int small_batches, const Emit& E, double* sum_w,
                                    double* sum_w2, HeadSmem& sm, uint32_t have = 0u, uint32_t blk = 0u,
                                    bool by_rule = false, int rule_blocks = 0) {
    const int tid = threadIdx.x;
    const int words = (hs.n + 31) >> 5;
    const uint32_t ns = (uint32_t)hs.n_s;
    if (c == 0) return 0;
    int flags = 0;
    const bool all = c >= ns;
    const bool invert = all || 2u * c > ns;
    const uint32_t target = all ? 0u : (invert ? ns - c : c);
    if (all) {
      // the whole residual: no draws; forget a batch that was generated ahead
      __syncthreads();
      for (int w = tid; w < words; w += NT) S.taken[w] = 0;
      __syncthreads();
    }
    int batches = blk > 0u ? 1 : 0;
    bool use_spec = have_spec;
    double aw = 0.0, aw2 = 0.0;
    const uint32_t rule = (uint32_t)(rule_blocks > 0 ? rule_blocks : first_blocks(small_batches, target));
    while (have < target) {
      if ((uint64_t)blk * 4ull >= (uint64_t)S.cap) break;
      DrawBatch B;
      if (use_spec) {
        B = spec;
        use_spec = false;
      } else {
        const uint32_t remaining = target - have;
        const int blocks = first_blocks(small_batches, remaining);
        make_batch(B, S, hs, blk, blocks, blk > 0, false, sm, (int)threadIdx.x);
      }
      ++batches;
      VATT_STAMP(S.dbg, 10);
      // accept in draw order: first proposals of residual tokens, until the target is reached
      const uint32_t acc = B.first & ~test_bits4(S.bm_f, B.tok);
      uint32_t total;
      uint32_t pos = block_exclusive_scan<NT>((uint32_t)__popc(acc), &total, sm.scan);
      const uint32_t room = target - have;
      VATT_STAMP(S.dbg, 11);
      // (written without nested per-draw branches: a divergent branch inside an unrolled loop serialises it)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool a = (acc >> e) & 1u;
        const bool take = a && pos < room;
        if (by_rule && take && pos + 1u == room) sm.last_block = blk + (uint32_t)tid;
        if (!invert) {
          if (take) emit_tok(E, have + pos, (int32_t)B.tok[e]);
          if (take && E.sc_dst && B.have_sc && have + pos < E.dst_cap) E.sc_dst[have + pos] = B.sc[e];
          if (sum_w) {
            const float sc = B.have_sc ? B.sc[e] : (take ? S.row[B.tok[e]] : 0.f);
            const double w = take ? (double)__expf(sc - S.m) : 0.0;
            aw += w;
            aw2 += w * w;
          }
        } else if (a && !take) {
          atomicAnd(&S.taken[B.tok[e] >> 5], ~(1u << (B.tok[e] & 31)));  // drawn after the sample was complete
        }
        pos += a ? 1u : 0u;
      }
      have += min(total, room);
      blk += (uint32_t)B.blocks;
      VATT_STAMP(S.dbg, 12);
    }
    if (!by_rule && batches > 1) flags |= 2;
    __syncthreads();
    if (by_rule && target > 0u && (have < target ? rule * 4u < S.cap : sm.last_block >= rule)) flags |= 2;
    if (have < target) {
      // draw cap reached: complete with the lowest-index residual tokens not yet accepted
      flags |= 4;
      const uint32_t need = target - have;
      for (int w = tid; w < words; w += NT) S.scratch[w] = mid_mask(hs, w) & ~S.bm_f[w] & ~S.taken[w];
      __syncthreads();
      word_prefix(S.scratch, words, S.wpre, sm);
      for (int w = tid; w < words; w += NT) {
        uint32_t bits = S.scratch[w];
        uint32_t pos = S.wpre[w];
        while (bits && pos < need) {
          const uint32_t i = (uint32_t)(w << 5) + (uint32_t)(__ffs(bits) - 1);
          bits &= bits - 1u;
          if (invert) {
            atomicOr(&S.taken[i >> 5], 1u << (i & 31));
          } else {
            emit_tok(E, have + pos, (int32_t)i);
            if (sum_w) {
              const double wt = (double)__expf(S.row[i] - S.m);
              aw += wt;
              aw2 += wt * wt;
            }
          }
          ++pos;
        }
      }
      __syncthreads();
      for (int w = tid; w < words; w += NT) S.scratch[w] = 0;
      __syncthreads();
    }
    if (invert) {
      // the sample is the residual minus the accepted tokens, in ascending order
      flags |= 1;
      for (int w = tid; w < words; w += NT) S.scratch[w] = mid_mask(hs, w) & ~S.bm_f[w] & ~S.taken[w];
      __syncthreads();
      word_prefix(S.scratch, words, S.wpre, sm);
      for (int w = tid; w < words; w += NT) {
        uint32_t bits = S.scratch[w];
        uint32_t pos = S.wpre[w];
        while (bits) {
          const int i = (w << 5) + (__ffs(bits) - 1);
          bits &= bits - 1u;
          emit_tok(E, pos, i);
          if (sum_w) {
            const double wt = (double)__expf(S.row[i] - S.m);
            aw += wt;
            aw2 += wt * wt;
          }
          ++pos;
        }
      }
      __syncthreads();
      for (int w = tid; w < words; w += NT) S.scratch[w] = 0;
      __syncthreads();
    }
    if (sum_w) {
      *sum_w += aw;
      *sum_w2 += aw2;
    }
    return flags;
  }

  // Rewrites a token list this workgroup wrote at dst (count distinct tokens below n) in ascending order:
  // the tokens are marked in the all-zero bitmap `scratch`, counted by bitmap word, and written back by
  // position; `scratch` is left all zero.  (An option of the plans: rows gathered in ascending order.)
  static __device__ void sort_ascending(int32_t* dst, uint32_t count, uint32_t* scratch, uint32_t* wpre, int n,
                                        HeadSmem& sm) {
    const int tid = threadIdx.x;
    const int words = (n + 31) >> 5;
    __syncthreads();  // the list is complete (global memory is coherent inside a workgroup)
    for (uint32_t t = tid; t < count; t += NT) mark_bit(scratch, (uint32_t)list_tok(dst, t, n));
    __syncthreads();
    word_prefix(scratch, words, wpre, sm);
    for (int w = tid; w < words; w += NT) {
      uint32_t bits = scratch[w];
      uint32_t pos = wpre[w];
      while (bits) {
        const int i = (w << 5) + (__ffs(bits) - 1);
        bits &= bits - 1u;
        if (pos < count) dst[pos] = i;
        ++pos;
      }
    }
    __syncthreads();
    for (int w = tid; w < words; w += NT) scratch[w] = 0;
    __syncthreads();
  }

  // Nested final sample (an option; Algorithm 1 draws the final sample afresh): the base sample, whose list
  // of b0 tokens this workgroup wrote at `base`, is kept as the head of the final sample, and the remaining
  // c - b0 tokens are drawn with the stream of S among the residual tokens outside the base sample.  The base
  // tokens are added to the bitmap of excluded tokens (bm, which S.bm_f points to) for that purpose.
  static __device__ __forceinline__ int draw_nested(const Sampler& S, HeadSizes hs, uint32_t b0, uint32_t c,
                                                    uint32_t* bm, const int32_t* base, int32_t* dst,
                                                    uint32_t dst_cap, int small_batches, HeadSmem& sm) {
    __syncthreads();  // the base list is complete (global memory is coherent inside a workgroup)
    for (uint32_t t = threadIdx.x; t < b0; t += NT) {
      const int tok = list_tok(base, t, hs.n);
      mark_bit(bm, (uint32_t)tok);
      if (t < dst_cap) dst[t] = tok;
    }
    __syncthreads();
    if (c <= b0 || dst_cap <= b0) return 0;
    hs.n_s -= (int)b0;
    const DrawBatch none = {};
    return draw_sample(S, hs, c - b0, none, false, small_batches, emit_to(dst + b0, dst_cap - b0), nullptr, nullptr, sm);
  }
};  // struct HeadOps

// Philox blocks of the batch that is generated ahead, before the top-k set is known: at most ahead_blocks, and of the
// stream of a sample that needs `most` accepted draws at most no more than it is likely to use.  While fewer than
// `most` of the n_s residual tokens are taken a draw from the L middle tokens is accepted with a probability of at
// least (n_s - most) / L, so `most` L / (n_s - most) draws suffice on average; six standard deviations are added (a
// batch that falls short costs time only).
template <int NT>
__host__ __device__ constexpr int ahead_blocks(int small_batches) {
  // (a workgroup of 1024 threads serves long rows, whose samples hold thousands of tokens)
  return small_batches ? kSmallBatchBlocks : (NT >= 1024 ? 1024 : NT < 256 ? NT : 256);
}
__device__ __forceinline__ int likely_blocks(int all, const HeadSizes& hs, int most) {
  const int L = max(hs.mid_hi - hs.mid_lo, 1);
  const float d = (float)most * (float)L / (float)max(hs.n_s - most, 1);
  return max(1, min(all, (int)((d + 6.f * sqrtf(d) + 19.f) * 0.25f)));
}
template <int NT>
__device__ __forceinline__ int ahead_blocks(int small_batches, const HeadSizes& hs, int most) {
  return likely_blocks(ahead_blocks<NT>(small_batches), hs, most);
}
// The most accepted draws the two samples can ask for: the smaller of the sample and its complement, the base sample
// being known and the final sample anything from the base sample up.
__device__ __forceinline__ int base_draws(const HeadSizes& hs) { return min(hs.b0, hs.n_s - hs.b0); }
__device__ __forceinline__ int final_draws(const HeadSizes& hs) { return hs.n_s / 2; }

// What a batch made ahead leaves of a thread's draws beside their tokens: ok (bits 0 - 3) and first (4 - 7) of DrawBatch, whether the
// batch was made at all (8), and its Philox blocks (16 - 31; only the caller-supplied path reads them, the scored path works them out).
__device__ __forceinline__ uint32_t pre_pack(const DrawBatch& B, bool made) {
  return (B.ok & 15u) | (B.first & 15u) << 4 | (made ? 256u : 0u) | (uint32_t)B.blocks << 16;
}
__device__ __forceinline__ bool pre_made_of(uint32_t f) { return (f & 256u) != 0u; }
__device__ __forceinline__ uint32_t pre_ok(uint32_t f) { return f & 15u; }
__device__ __forceinline__ uint32_t pre_first(uint32_t f) { return f >> 4 & 15u; }
__device__ __forceinline__ int pre_blocks(uint32_t f) { return (int)(f >> 16); }

// ---------------------------------------------------------------------------
// The first batch of draws of one sampler stream of one (sequence, head), with repeated tokens resolved, made
// ahead of the selection kernel: the draw sequences depend on the seed, the head and the sequence length only,
// not on the scores, so workgroups of the score launch make them while the others stream K.  The selection
// kernel (512 threads: the lower half owns stream 0, the upper half stream 1) then starts from these batches.
// ---------------------------------------------------------------------------
struct PreArgs {
  const int32_t* seq_lens;
  const uint64_t* seq_seeds;
  uint4* pre_tok;       // [B*Hq][512]: the four proposed tokens of every thread of the selection kernel
  uint32_t* pre_flags;  // [B*Hq][512]: see pre_pack
  SelectParams sp;
  int n_max, Hq, small_batches;
  uint32_t draw_cap;
  int job_rows;  // rows of the score grid that make batches instead of scores (0: none)
};

constexpr int kPreThreads = 256;  // workgroup size of a job: the score kernel's

// LDS layout of a job: HeadSmem, then two bitmaps of words_max words (drawn tokens, scratch) and the mail slots.
__host__ __device__ inline size_t prework_lds_bytes(int n_max) {
  const size_t words_max = (size_t)bitmap_words(n_max);
  return ((sizeof(HeadOps<kPreThreads>::HeadSmem) + 15) & ~size_t(15)) + (2 * words_max + kMailSlots) * sizeof(uint32_t);
}

__device__ __forceinline__ void prework_job(const PreArgs& A, int b, int h, int stream, unsigned char* smem) {
  constexpr int NT = kPreThreads;
  using O = HeadOps<NT>;
  const int tid = threadIdx.x, bh = b * A.Hq + h;
  const int n = max(min(max(A.seq_lens[b], 1), A.n_max), 1);
  const HeadSizes hs = head_sizes(n, A.sp);
  const int words_max = bitmap_words(A.n_max);
  const int words = (n + 31) >> 5;
  O::HeadSmem& sm = *reinterpret_cast<O::HeadSmem*>(smem);
  uint32_t* taken = reinterpret_cast<uint32_t*>(smem + ((sizeof(O::HeadSmem) + 15) & ~size_t(15)));
  uint32_t* scratch = taken + words_max;
  uint32_t* mail = scratch + words_max;
  for (int w = tid; w < words; w += NT) {
    taken[w] = 0;
    scratch[w] = 0;
  }
  __syncthreads();
  const uint32_t L = (uint32_t)max(hs.mid_hi - hs.mid_lo, 1);
  O::Sampler S;
  S.taken = taken;
  S.scratch = scratch;
  S.mail = mail;
  S.bm_f = nullptr;
  S.wpre = nullptr;
  S.row = nullptr;
  S.seed = A.seq_seeds[b];
  S.stream = (uint32_t)stream;
  S.head = (uint32_t)h;
  S.query = 0u;
  S.L = L;
  S.thr = (uint32_t)((0x100000000ull - (uint64_t)L) % (uint64_t)L);
  {
    const uint64_t dflt = 64ull * (uint64_t)L + 4096ull;
    S.cap = (uint32_t)min(A.draw_cap ? (uint64_t)A.draw_cap : dflt, 0x80000000ull);
  }
  S.m = 0.f;
  S.dbg = nullptr;
  // (what the 512-thread selection kernel asks for)
  const int blocks = ahead_blocks<2 * NT>(A.small_batches, hs, stream == 0 ? base_draws(hs) : final_draws(hs));
  const bool make = hs.n_s > 0 && hs.b0 < hs.n_s && blocks <= NT;
  DrawBatch mine = {};
  if (make) O::make_batch(mine, S, hs, 0u, blocks, false, false, sm, tid);
  const int64_t at = (int64_t)bh * (2 * NT) + stream * NT + tid;
  A.pre_tok[at] = make_uint4(mine.tok[0], mine.tok[1], mine.tok[2], mine.tok[3]);
  A.pre_flags[at] = pre_pack(mine, make);
}

}  // namespace vatt
