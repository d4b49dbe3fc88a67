// Dense decode attention (Eq. 1) on the same cache, and the KV append.
#include "vatt_internal.h"

namespace vatt {
namespace {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc,
                                         false);
}

constexpr float kNegBig = -1.0e30f;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
// The upper (lower) 16 bits of two words, those of `a` in the lower half.
__device__ __forceinline__ uint32_t upper_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ uint32_t lower_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }

// 16 bytes of a K or V row; STREAM: nobody else reads them
template <bool STREAM>
__device__ __forceinline__ uint4 dense_load_16(const uint16_t* p) {
  return STREAM ? load_stream_16(p) : *reinterpret_cast<const uint4*>(p);
}

// Column c of row i (contiguous cache: a uniform address and 32-bit offsets, for at most 170752 tokens, take fewest
// registers).
template <int D, bool PAGED>
__device__ __forceinline__ const uint16_t* dense_row(const uint16_t* base, const KVLayout& L, int seq, int kvh, int i, int blk, int c) {
  if constexpr (PAGED) return base + kv_row_offset_in<true>(L, seq, kvh, i, blk) + c;
  else return base + kv_row_offset<false>(L, seq, kvh, 0) + (uint32_t)(i * D + c);
}

struct DenseArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  KVLayout Lk, Lv;
  const int32_t* seq_lens;
  float* part;     // [B * q_len * Hq][splits][d]: partial sums of the weighted V rows
  float2* part_ml;  // [B * q_len * Hq][splits]: (max, sum of the weights); the unused ones of a row come last, max -inf
  int2* keys;       // [B][splits]: keys (from, up to) of a sequence's pieces, left by dense_kernel
  float* out_o;
  float* out_lse;
  int batch, n_max, Hq;
  int splits;  // most partials a row of the output can have
  int share;   // > 0: the keys of all sequences are dealt out evenly to this many workgroups per KV head and round;
               // 0: every sequence is cut into `splits` equal ranges
  int q_len;   // query tokens per sequence
  int rounds;  // workgroups that take the same keys because their query vectors do not fit one
  float sm_scale;
};

// How the keys of a batch are dealt out to the workgroups of a KV head.  The sequences' lengths in units of `unit`
// keys are laid end to end and cut into runs, one per workgroup, so that ragged lengths leave no workgroup with more
// than its share.  A run may hold the end of one sequence and the beginning of the next, at the price of draining and
// refilling the workgroup's pipeline (about 2 us per further sequence).  Where that is not worth it (the sequences,
// each rounded up to whole runs, need no more workgroups anyway, or a run is short) every sequence starts a new run:
// 9 x 14846 tokens 61 us in whole runs, 52 us end to end; 8 x 0.2K .. 4K tokens 14.4 and 17.4 us.  The partial sums of
// a sequence are numbered from its first run on.  A wave-wide computation (all lanes active) that every workgroup
// makes for itself, 64 sequences at a time.
struct DenseDeal {
  uint32_t run;       // units per workgroup
  bool whole;         // every sequence starts a new run
  int b0;             // first of the 64 sequences at hand
  uint32_t before;    // units laid out before it
  int n;              // this lane's sequence: length (0 beyond the last), and units laid out up to its end
  uint32_t u, incl;
};
__device__ __forceinline__ int dense_length(const DenseArgs& A, int b) {
  return b < A.batch ? min(max(A.seq_lens[b], 1), A.n_max) : 0;
}
__device__ __forceinline__ void dense_lay_out(DenseDeal& d) {
  const uint32_t laid = d.whole ? (d.u + d.run - 1) / d.run * d.run : d.u;
  d.incl = d.before + wave_inclusive_scan_u32(laid);
}
template <int UNIT, int ROW_BYTES>
__device__ __forceinline__ DenseDeal dense_deal(const DenseArgs& A) {
  constexpr uint32_t kShortRun = 384 * 1024 / (2 * ROW_BYTES * UNIT);  // units: 384 KB of K and V
  DenseDeal d;
  d.b0 = 0;
  d.before = 0;
  d.n = dense_length(A, (int)(threadIdx.x & 63));
  d.u = (uint32_t)(d.n + UNIT - 1) / UNIT;
  auto units = [&](int b0) {
    return b0 == 0 ? d.u : (uint32_t)(dense_length(A, b0 + (int)(threadIdx.x & 63)) + UNIT - 1) / UNIT;
  };
  uint32_t total = 0, longest = 0, whole_runs = 0;
  for (int b0 = 0; b0 < A.batch; b0 += kWave) {
    const uint32_t u = units(b0);
    total += wave_sum_u32(u);
    longest = max(longest, wave_max_u32(u));
  }
  d.run = (total + (uint32_t)A.share - 1) / (uint32_t)A.share;
  // (a sequence has at most A.splits partial sums, and may touch one run more than its length fills, but not more than it
  // has units)
  if (longest > (uint32_t)A.splits && longest > d.run * (uint32_t)(A.splits - 1)) d.run = (longest + (uint32_t)A.splits - 2) / (uint32_t)(A.splits - 1);
  d.whole = d.run <= kShortRun;
  if (!d.whole) {
    for (int b0 = 0; b0 < A.batch; b0 += kWave) whole_runs += wave_sum_u32((units(b0) + d.run - 1) / d.run);
    d.whole = whole_runs <= (uint32_t)A.share;
  }
  dense_lay_out(d);
  return d;
}

// Dense attention with the query vectors of a KV head on the matrix cores: every K and V row is read from HBM
// once for all query tokens of the sequence and all heads of the group.  Query vector c = t * G + g (query token
// t, head g of the group) is a column of two products over 32 keys at a time,
//   S [keys x vectors] = K Q^T   and   O^T [d x vectors] += V^T P^T,   P = exp(S - m),
// both v_mfma_f32_16x16x32_bf16 (operand lane l: row or column l % 16, eight inner elements; result lane l: column
// l % 16, rows 4 (l / 16) .. + 3).
//   * The result layout of S is, with the inner index of the second product numbered to suit, its operand layout
//     for P: lane group g = l / 16 holds keys 4 g + r and 16 + 4 g + r as inner elements r and 4 + r.
//   * V needs no transposition through LDS: lane (g, i) loads d / 16 consecutive values of the eight rows of group
//     g, which makes whole 256-byte rows per 16 lanes, and pairs them by rows in registers; row i of operand e
//     is then column (d / 16) i + e of V.
//   * P goes in as three bf16 terms (leading, next, last eight bits of the fp32 value), which add up to it exactly:
//     the products and sums keep fp32 accuracy.
//   * K rows pass through an LDS tile of the wave, as in the multi-query score kernel.
// The running maximum of a column moves only when a score exceeds it by more than kLazy (a wave-uniform branch
// that is rarely taken after the first rows); until then weights may exceed 1, by at most exp(kLazy).
// What bounds it: the stream of K and V (2 * Hkv * n * d * 2 bytes per sequence), and from 64 query vectors on also the
// vector instructions of exp and of splitting the weights.  One wave has one step's 16 KB in flight: K is requested
// as soon as the last K rows are in the LDS tile, V as soon as the last V rows are used.  Measured against dot products
// with one scan of the cache per query token: 4 x 32K tokens (77 us at 7 TB/s) with 1 / 2 / 4 / 8 query tokens 93 /
// 146 / 271 / 528 -> 88 / 87 / 88 / 90 us; 1 x 32K with 16 query tokens 267 -> 43 us; 16 x 32K 350 -> 312 us;
// 32 ragged sequences on 16-token pages 250 -> 180 us.
// A workgroup's four waves are WQ groups of 16 NQT query vectors times 4 / WQ key ranges; waves with the same
// key range read the same rows at about the same time (plain loads, so that the L1 and L2 serve the repeats).
template <int D, bool PAGED, int NQT, int WQ>
__global__ __launch_bounds__(kDenseThreads, 2) void dense_kernel(DenseArgs A) {
  constexpr int S = D / 32;         // MFMA steps over a row of K
  constexpr int E = D / 16;         // values of a V row per lane = MFMA tiles over the head dimension
  constexpr int LPR = D / 8;        // lanes per K row load
  constexpr int RPI = kWave / LPR;  // K rows per wave instruction
  constexpr int KL = kDenseKeys / RPI;
  constexpr int WAVES = kDenseThreads / kWave, WK = WAVES / WQ;
  constexpr float kLazy = 6.0f;
  constexpr float kLog2e = 1.44269504088896340736f;

  // (the wave's number as a scalar: its key range and the loop over it then take no vector registers, of which there are
  // none to spare at 128 columns; at 64 a workgroup alone with 8K tokens takes 64 us with it and 63 without)
  const int tid = threadIdx.x, lane = tid & 63, wave = D == 128 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int i16 = lane & 15, g4 = lane >> 4, lrow = lane / LPR, lchunk = lane % LPR;
  const int wq = wave % WQ, wk = wave / WQ;
  constexpr int kUnit = kDenseKeys * WK;
  const int kvh = blockIdx.x, slot = (int)blockIdx.y / A.rounds, round = (int)blockIdx.y - slot * A.rounds;
  const int G = A.Hq / (int)gridDim.x, Q = A.q_len, QG = Q * G;
  const int c_base = (round * WQ + wq) * 16 * NQT;

  union Lds {
    uint4 k[WAVES][kDenseKeys * (LPR + 1)];  // K tile of each wave; rows one chunk apart in the banks
    float4 o[WAVES][4][E / 4][kWave];        // sums of one 16-vector tile of every wave, for the merge at the end
  };
  __shared__ Lds lds;
  __shared__ float s_m[WAVES][16], s_l[WAVES][16];
  uint4* kt = lds.k[wave];

  DenseDeal deal = {};
  uint32_t at = 0, at_end = 1;
  if (A.share) {
    deal = dense_deal<kUnit, 2 * D>(A);
    at = (uint32_t)slot * deal.run;
    at_end = at + deal.run;
  }
  while (at < at_end) {
  int seq, n, split, u_lo, u_n, idle = 0;  // this workgroup's next piece of a sequence, in units
  if (A.share) {
    uint64_t here;
    while ((here = __ballot(deal.incl > at)) == 0) {
      if (deal.b0 + kWave >= A.batch) return;  // beyond the last sequence (the same in every wave)
      deal.b0 += kWave;
      deal.before = (uint32_t)__builtin_amdgcn_readlane((int)deal.incl, 63);
      deal.n = dense_length(A, deal.b0 + lane);
      deal.u = (uint32_t)(deal.n + kUnit - 1) / kUnit;
      dense_lay_out(deal);
    }
    const int l = __ffsll((unsigned long long)here) - 1;
    const uint32_t begin = l ? (uint32_t)__builtin_amdgcn_readlane((int)deal.incl, l - 1) : deal.before;
    const uint32_t end = begin + (uint32_t)__builtin_amdgcn_readlane((int)deal.u, l);
    seq = deal.b0 + l;
    n = __builtin_amdgcn_readlane(deal.n, l);
    split = slot - (int)(begin / deal.run);
    u_lo = (int)(at - begin);
    u_n = (int)(min(end, at_end) - at);
    // the last piece of a sequence also marks the places of partial sums that the sequence has no pieces for
    if (end <= at_end) idle = A.splits - 1 - split;
    at = deal.whole ? at_end : end;
  } else {
    seq = blockIdx.z;
    split = slot;
    n = dense_length(A, seq);
    u_n = ((n + kUnit - 1) / kUnit + A.splits - 1) / A.splits;
    u_lo = split * u_n;
    at = at_end;
  }
  const int blk_hi = min((u_lo + u_n) * kUnit, n);
  // (the same for every KV head and round)
  if (kvh == 0 && round == 0 && tid == 0) A.keys[seq * A.splits + split] = make_int2(u_lo * kUnit, blk_hi);
  const int lo = min(u_lo * kUnit + wk * u_n * kDenseKeys, n), hi = min(lo + u_n * kDenseKeys, blk_hi);

  uint4 bq[NQT][S];
  int seen[NQT];  // tokens the query of this lane's column sees
#pragma unroll
  for (int nt = 0; nt < NQT; ++nt) {
    const int c = min(c_base + nt * 16 + i16, QG - 1);  // (columns beyond the last vector repeat it and are not stored)
    const int t = c / G, g = c - t * G;
    const uint16_t* src = A.q + (((int64_t)seq * Q + t) * A.Hq + (int64_t)kvh * G + g) * D + g4 * 8;
#pragma unroll
    for (int s = 0; s < S; ++s) bq[nt][s] = *reinterpret_cast<const uint4*>(src + s * 32);
    seen[nt] = max(n - (Q - 1 - t), 1);
  }
  f32x4_t acc[NQT][E];
  float mrun[NQT], lrun[NQT];
#pragma unroll
  for (int nt = 0; nt < NQT; ++nt) {
    mrun[nt] = kNegBig;
    lrun[nt] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[nt][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  uint4 kr[KL];
  uint32_t vr[8][E / 2];
  auto row = [&](const uint16_t* base, const KVLayout& L, int i, int blk, int c) {
    return dense_row<D, PAGED>(base, L, seq, kvh, i, blk, c);
  };
  // (paged cache: the block-table entries of all rows first, so that no row waits for the entry of the one before)
  auto load_k = [&](int i0) {
    int blk[KL];
    auto key = [&](int u) { return min(i0 + u * RPI + lrow, hi - 1); };
#pragma unroll
    for (int u = 0; u < KL; ++u) blk[u] = kv_block<PAGED>(A.Lk, seq, key(u));
#pragma unroll
    for (int u = 0; u < KL; ++u) kr[u] = dense_load_16<WQ == 1>(row(A.k, A.Lk, key(u), blk[u], lchunk * 8));
  };
  auto load_v = [&](int i0) {
    int blk[8];
    auto key = [&](int j) { return min(i0 + (j < 4 ? 0 : 12) + 4 * g4 + j, hi - 1); };
#pragma unroll
    for (int j = 0; j < 8; ++j) blk[j] = kv_block<PAGED>(A.Lv, seq, key(j));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t* src = row(A.v, A.Lv, key(j), blk[j], i16 * E);
      if constexpr (D == 128) {
        const uint4 x = dense_load_16<WQ == 1>(src);
        vr[j][0] = x.x; vr[j][1] = x.y; vr[j][2] = x.z; vr[j][3] = x.w;
      } else {
        const uint2 x = *reinterpret_cast<const uint2*>(src);
        vr[j][0] = x.x; vr[j][1] = x.y;
      }
    }
  };
  if (lo < hi) {
    load_k(lo);
    load_v(lo);
  }
  for (int i0 = lo; i0 < hi; i0 += kDenseKeys) {
    // K rows into the tile, the next ones requested, the scores of 32 keys
#pragma unroll
    for (int u = 0; u < KL; ++u) kt[(u * RPI + lrow) * (LPR + 1) + lchunk] = kr[u];
    load_k(i0 + kDenseKeys);
    __builtin_amdgcn_wave_barrier();
    f32x4_t sc[NQT][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      uint4 ka[S];
#pragma unroll
      for (int s = 0; s < S; ++s) ka[s] = kt[(t * 16 + i16) * (LPR + 1) + s * 4 + g4];
#pragma unroll
      for (int nt = 0; nt < NQT; ++nt) {
        sc[nt][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s)
          sc[nt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[s]),
                                                              __builtin_bit_cast(bf16x8_t, bq[nt][s]), sc[nt][t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
    const bool edge = i0 + kDenseKeys > min(hi, n - Q + 1);  // some column does not see all of the 32 keys
    uint4 pb[NQT][3];
#pragma unroll
    for (int nt = 0; nt < NQT; ++nt) {
      float s[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] = sc[nt][j >> 2][j & 3] * A.sm_scale;
      const int end = min(hi, seen[nt]) - i0 - 4 * g4;  // key j of this lane counts when its offset is below this
      if (edge) {
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] = (j < 4 ? 0 : 12) + j < end ? s[j] : kNegBig;
      }
      float top = s[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) top = fmaxf(top, s[j]);
      if (__ballot(top > mrun[nt] + kLazy)) {
        top = fmaxf(top, __shfl_xor(top, 16));
        top = fmaxf(top, __shfl_xor(top, 32));
        const float mnew = fmaxf(mrun[nt], top);
        const float alpha = __expf(mrun[nt] - mnew);
        mrun[nt] = mnew;
        lrun[nt] *= alpha;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[nt][e] *= alpha;
      }
      uint32_t w[3][8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float p = __builtin_amdgcn_exp2f((s[j] - mrun[nt]) * kLog2e);
        if (edge) p = (j < 4 ? 0 : 12) + j < end ? p : 0.f;
        lrun[nt] += p;
        const float r1 = p - __uint_as_float(__float_as_uint(p) & 0xffff0000u);
        const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
        w[0][j] = __float_as_uint(p);
        w[1][j] = __float_as_uint(r1);
        w[2][j] = __float_as_uint(r2);
      }
#pragma unroll
      for (int x = 0; x < 3; ++x)
        pb[nt][x] = make_uint4(upper_halves(w[x][0], w[x][1]), upper_halves(w[x][2], w[x][3]),
                               upper_halves(w[x][4], w[x][5]), upper_halves(w[x][6], w[x][7]));
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      uint32_t a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        a[j] = (e & 1) ? upper_halves(vr[2 * j][e / 2], vr[2 * j + 1][e / 2]) : lower_halves(vr[2 * j][e / 2], vr[2 * j + 1][e / 2]);
      const uint4 va = make_uint4(a[0], a[1], a[2], a[3]);
#pragma unroll
      for (int nt = 0; nt < NQT; ++nt) {
#pragma unroll
        for (int x = 2; x >= 0; --x)
          acc[nt][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, va),
                                                               __builtin_bit_cast(bf16x8_t, pb[nt][x]), acc[nt][e], 0, 0, 0);
      }
    }
    load_v(i0 + kDenseKeys);
  }

  // Log-sum-exp merge of the waves' key ranges, one 16-vector tile of every wave at a time.  The sums stay in
  // the result layout throughout: wave wk finishes the result rows 4 g + r of its share of the r, which it reads
  // from every wave with the same vectors, and stores the E consecutive columns of each.
  constexpr int RW = 4 / WK;  // rows r per wave
#pragma unroll
  for (int nt = 0; nt < NQT; ++nt) {
    float l = lrun[nt];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    float m = mrun[nt], fac[WK];
    fac[0] = 1.f;
    if constexpr (WK > 1) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int e = 0; e < E; e += 4)
          lds.o[wave][r][e / 4][lane] = make_float4(acc[nt][e][r], acc[nt][e + 1][r], acc[nt][e + 2][r], acc[nt][e + 3][r]);
      }
      if (g4 == 0) {
        s_m[wave][i16] = m;
        s_l[wave][i16] = l;
      }
      __syncthreads();
      l = 0.f;
#pragma unroll
      for (int w = 0; w < WK; ++w) m = fmaxf(m, s_m[w * WQ + wq][i16]);
#pragma unroll
      for (int w = 0; w < WK; ++w) {
        fac[w] = __expf(s_m[w * WQ + wq][i16] - m);
        l += s_l[w * WQ + wq][i16] * fac[w];
      }
    }
    const int c = c_base + nt * 16 + i16;
    const int tok = c / G, g = c - tok * G;
    const int64_t place = (((int64_t)seq * Q + tok) * A.Hq + (int64_t)kvh * G + g) * A.splits + split;
    float* part = A.part + place * D;
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const int r = wk * RW + rr;
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        float4 o;
        if constexpr (WK > 1) {
          o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int w = 0; w < WK; ++w) {
            const float4 x = lds.o[w * WQ + wq][r][e / 4][lane];
            o.x += x.x * fac[w];
            o.y += x.y * fac[w];
            o.z += x.z * fac[w];
            o.w += x.w * fac[w];
          }
        } else {
          o = make_float4(acc[nt][e][rr], acc[nt][e + 1][rr], acc[nt][e + 2][rr], acc[nt][e + 3][rr]);
        }
        if (c < QG) *reinterpret_cast<float4*>(part + E * (4 * g4 + r) + e) = o;
      }
    }
    if (c < QG && wk == 0) {
      for (int x = g4; x <= idle; x += 4) A.part_ml[place + x] = x == 0 ? make_float2(m, l) : make_float2(-INFINITY, 0.f);
    }
  }
  if (at < at_end) {
    deal.n = dense_length(A, deal.b0 + lane);  // (read again rather than kept in registers across the keys)
    deal.u = (uint32_t)(deal.n + kUnit - 1) / kUnit;
    dense_lay_out(deal);
    if (WK > 1) __syncthreads();  // the next piece's K tiles take the place of the sums
  }
  }
}

// One or two query vectors per KV head (single-token steps without or with little grouping), which would leave the
// matrix cores' 16 columns empty: dot products.  A workgroup owns a range of a sequence's keys; each wave walks a
// quarter of it with the lane layout of the score pass, keeping a running (max, sum, accumulator) per lane group, and
// needs few enough registers for 16 waves per CU.  At d = 64: 16 x 9768 tokens on pages 101 us against 115 us of
// dense_kernel, 4 x 25K ragged 38 against 42 us; with 4 vectors per KV head dense_kernel is ahead (57 against 62 us).
template <int D, int G, bool PAGED>
__global__ __launch_bounds__(kDenseThreads) void dense_dot_kernel(DenseArgs A) {
  constexpr int LPR = D / 8;
  constexpr int RPW = kWave / LPR;
  constexpr int WAVES = kDenseThreads / kWave;
  constexpr int U = 4;

  const int kvh = blockIdx.x;
  const int split = blockIdx.y, seq = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, rsub = lane / LPR;
  const int n = min(max(A.seq_lens[seq], 1), A.n_max);
  // key range of this workgroup, then of this wave (multiples of RPW * U rows except at the end)
  const int step = RPW * U;
  const int per_blk = ((n + A.splits - 1) / A.splits + step * WAVES - 1) / (step * WAVES) * (step * WAVES);
  const int blk_lo = split * per_blk, blk_hi = min(blk_lo + per_blk, n);
  const int per_wave = per_blk / WAVES;
  const int lo = blk_lo + wave * per_wave, hi = min(lo + per_wave, blk_hi);

  uint32_t qw[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 t = *reinterpret_cast<const uint4*>(A.q + ((int64_t)seq * A.Hq + (int64_t)kvh * G + g) * D + sub * 8);
    qw[g][0] = t.x;
    qw[g][1] = t.y;
    qw[g][2] = t.z;
    qw[g][3] = t.w;
  }
  float mrun[G], lrun[G], acc[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    mrun[g] = kNegBig;
    lrun[g] = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[g][c] = 0.f;
  }

  for (int i0 = lo; i0 < hi; i0 += step) {
    uint4 kk[U], vv[U];
    bool ok[U];
    int blk[U];
    // (paged cache: the block-table entries of all rows first, outside the test on the row index, so that no
    // row waits for the entry of the one before; K and V share the table)
#pragma unroll
    for (int u = 0; u < U; ++u) blk[u] = kv_block<PAGED>(A.Lk, seq, min(i0 + u * RPW + rsub, hi - 1));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * RPW + rsub;
      ok[u] = i < hi;
      kk[u] = vv[u] = make_uint4(0u, 0u, 0u, 0u);
      if (ok[u]) {
        const uint16_t* pk = A.k + kv_row_offset_in<PAGED>(A.Lk, seq, kvh, i, blk[u]) + sub * 8;
        const uint16_t* pv = A.v + kv_row_offset_in<PAGED>(A.Lv, seq, kvh, i, blk[u]) + sub * 8;
        kk[u] = load_stream_16(pk);
        vv[u] = load_stream_16(pv);
      }
    }
    float s[G][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float a = 0.f;
        a = dot2_bf16(kk[u].x, qw[g][0], a);
        a = dot2_bf16(kk[u].y, qw[g][1], a);
        a = dot2_bf16(kk[u].z, qw[g][2], a);
        a = dot2_bf16(kk[u].w, qw[g][3], a);
        a = group_sum<LPR>(a);
        s[g][u] = ok[u] ? a * A.sm_scale : kNegBig;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mnew = mrun[g];
#pragma unroll
      for (int u = 0; u < U; ++u) mnew = fmaxf(mnew, s[g][u]);
      const float alpha = __expf(mrun[g] - mnew);
      mrun[g] = mnew;
      lrun[g] *= alpha;
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[g][c] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float p = ok[u] ? __expf(s[g][u] - mnew) : 0.f;
        lrun[g] += p;
        const uint32_t ww[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          acc[g][2 * c] += p * bf16_lo(ww[c]);
          acc[g][2 * c + 1] += p * bf16_hi(ww[c]);
        }
      }
    }
  }

  // merge the lane groups of the wave
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float mall = mrun[g];
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) mall = fmaxf(mall, __shfl_xor(mall, o));
    const float sc = __expf(mrun[g] - mall);
    lrun[g] *= sc;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[g][c] *= sc;
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) {
      lrun[g] += __shfl_xor(lrun[g], o);
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[g][c] += __shfl_xor(acc[g][c], o);
    }
    mrun[g] = mall;
  }
  __shared__ float s_acc[WAVES][G][D];
  __shared__ float s_m[WAVES][G], s_l[WAVES][G];
  if (rsub == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int c = 0; c < 8; ++c) s_acc[wave][g][sub * 8 + c] = acc[g][c];
      if (sub == 0) {
        s_m[wave][g] = mrun[g];
        s_l[wave][g] = lrun[g];
      }
    }
  }
  __syncthreads();
  for (int t = tid; t < G * D; t += kDenseThreads) {
    const int g = t / D, c = t % D;
    float mall = s_m[0][g];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) mall = fmaxf(mall, s_m[w][g]);
    float a = 0.f, l = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float sc = __expf(s_m[w][g] - mall);
      a += s_acc[w][g][c] * sc;
      l += s_l[w][g] * sc;
    }
    const int64_t place = ((int64_t)seq * A.Hq + (int64_t)kvh * G + g) * A.splits + split;
    A.part[place * D + c] = a;
    if (c == 0) A.part_ml[place] = make_float2(blk_lo < n ? mall : -INFINITY, l);
  }
}

// Keys lo .. hi - 1 again for query vector bh, by the whole workgroup of dense_merge_kernel: dot products and a running
// maximum per lane group, every row only where it is seen.  The sums go where dense_kernel would have left them.
template <int D, bool PAGED>
__device__ __forceinline__ void dense_again(const DenseArgs& A, int64_t bh, int seq, int kvh, int lo, int hi, float* part, float2* part_ml) {
  constexpr int LPR = D / 8, RPW = kWave / LPR, WAVES = 2 * D / kWave, U = 4;
  __shared__ float s_acc[WAVES][D], s_m[WAVES], s_l[WAVES];
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // (nothing of this is worked out ahead: the merge has no registers to spare for it)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), sub = lane % LPR, rsub = lane / LPR;
  const uint4 qv = *reinterpret_cast<const uint4*>(A.q + bh * D + sub * 8);
  float m = kNegBig, l = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int i0 = lo + wave * RPW * U + rsub; i0 - rsub < hi; i0 += WAVES * RPW * U) {
    int blk[U];
    uint4 kk[U], vv[U];
    auto key = [&](int u) { return min(i0 + u * RPW, hi - 1); };
#pragma unroll
    for (int u = 0; u < U; ++u) blk[u] = kv_block<PAGED>(A.Lk, seq, key(u));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      kk[u] = *reinterpret_cast<const uint4*>(dense_row<D, PAGED>(A.k, A.Lk, seq, kvh, key(u), blk[u], sub * 8));
      vv[u] = *reinterpret_cast<const uint4*>(dense_row<D, PAGED>(A.v, A.Lv, seq, kvh, key(u), blk[u], sub * 8));
    }
    float s[U], mnew = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = dot2_bf16(kk[u].x, qv.x, 0.f);
      s[u] = dot2_bf16(kk[u].y, qv.y, s[u]);
      s[u] = dot2_bf16(kk[u].z, qv.z, s[u]);
      s[u] = group_sum<LPR>(dot2_bf16(kk[u].w, qv.w, s[u])) * A.sm_scale;
      mnew = fmaxf(mnew, s[u]);  // (a row beyond the range repeats the last one)
    }
    const float alpha = __expf(m - mnew);
    m = mnew;
    l *= alpha;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * RPW < hi) {
        const float p = __expf(s[u] - m);
        const uint32_t ww[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
        l += p;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          acc[2 * c] += p * bf16_lo(ww[c]);
          acc[2 * c + 1] += p * bf16_hi(ww[c]);
        }
      }
    }
  }
  float mall = m;
#pragma unroll
  for (int o = LPR; o < kWave; o <<= 1) mall = fmaxf(mall, __shfl_xor(mall, o));
  const float f = __expf(m - mall);
  l *= f;
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] *= f;
#pragma unroll
  for (int o = LPR; o < kWave; o <<= 1) {
    l += __shfl_xor(l, o);
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += __shfl_xor(acc[c], o);
  }
  if (rsub == 0) {
#pragma unroll
    for (int c = 0; c < 8; ++c) s_acc[wave][sub * 8 + c] = acc[c];
  }
  if (lane == 0) {
    s_m[wave] = mall;
    s_l[wave] = l;
  }
  __syncthreads();
  float M = s_m[0], a = 0.f, lt = 0.f;
#pragma unroll
  for (int w = 1; w < WAVES; ++w) M = fmaxf(M, s_m[w]);
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const float g = __expf(s_m[w] - M);
    a += s_acc[w][tid % D] * g;
    lt += s_l[w] * g;
  }
  if (tid < D) part[tid] = a;
  if (tid == 0) *part_ml = make_float2(M, lt);
  __syncthreads();
}

// Log-sum-exp merge of the partial sums of one head.  Bound by the latency of two dependent loads: every wave loads
// the (max, sum) pairs for itself, one (or two) per lane, so that the weights of the partial sums are a wave-wide
// reduction and no barrier; two halves of the workgroup take alternate partial sums so that their loads are in
// flight together, and the first ones are requested before it is known how many there are.
// AGAIN (after dense_kernel): V rows with an Inf or a NaN.  The second product there gives every column every V row of a
// step, with weight 0 where the column does not see the token, and in three terms of which some are 0: such a row makes a
// NaN where it has no say (0 x Inf), which stays in the sums.  Finding it here costs dense_kernel nothing; the pieces with
// an Inf or a NaN are then taken again for this head alone.  With such a row in every sequence, 4 x 32K tokens with 1 / 8
// query tokens take 227 / 244 us instead of 87 / 89.  (A second loop in dense_kernel instead took so many registers that
// those 89 us became 105.  Written as a loop around the merge, or with more than 64 registers, this kernel took 7.6 instead of
// 4.8 us for 96 rows of 32 heads.)
template <int D, bool PAGED, bool AGAIN>
__global__ __launch_bounds__(2 * D, 8) void dense_merge_kernel(DenseArgs A, int Hkv) {
  static_assert(kDenseSplitsMax == 2 * kWave, "two pairs per lane");
  constexpr int kAhead = 4, WAVES = 2 * D / kWave;
  // blockIdx.x runs over the KV heads first, then over the heads of a group (as in the dense kernel's grid)
  const int h = head_of_block((int)blockIdx.x, A.Hq, Hkv, 1), b = blockIdx.y;
  const int64_t bh = (int64_t)b * A.Hq + h;
  const int c = threadIdx.x % D, half = threadIdx.x / D, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* p = A.part + bh * A.splits * D;
  float2* ml = A.part_ml + bh * A.splits;
  const float2 none = make_float2(-INFINITY, 0.f);
  __shared__ float s_a[D];
  __shared__ int s_odd[WAVES];
  float a, l, mall;
  int splits;
  auto combine = [&]() __attribute__((always_inline)) {  // (ends with a barrier; whether this half's sum is finite goes to s_odd)
    const float2 x0 = lane < A.splits ? ml[lane] : none, x1 = kWave + lane < A.splits ? ml[kWave + lane] : none;
    float first[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) first[u] = p[min(half + 2 * u, A.splits - 1) * D + c];
    // (unused ones come last; a piece all of whose scores are -inf has the maximum kNegBig)
    splits = (int)(__popcll(__ballot(x0.x > -INFINITY)) + __popcll(__ballot(x1.x > -INFINITY)));
    mall = wave_max(fmaxf(x0.x, x1.x));
    const float w0 = __expf(x0.x - mall), w1 = __expf(x1.x - mall);
    l = wave_sum_f32(x0.y * w0 + x1.y * w1);
    auto weight = [&](int s) {
      return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s < kWave ? w0 : w1), s & (kWave - 1)));
    };
    a = 0.f;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int s = half + 2 * u;
      if (s < splits) a += first[u] * weight(s);
    }
    for (int s = half + 2 * kAhead; s < splits; s += 2) a += p[s * D + c] * weight(s);
    if (half == 1) s_a[c] = a;
    if (AGAIN) {
      const uint64_t odd = __ballot(!(fabsf(a) < INFINITY));
      if (lane == 0) s_odd[wave] = odd != 0;
    }
    __syncthreads();
  };
  combine();
  if constexpr (AGAIN) {
    int odd = s_odd[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) odd |= s_odd[w];
    if (__builtin_amdgcn_readfirstlane(odd)) {
      const int seq = seq_of_pair(b, A.q_len), t = b - seq * A.q_len;
      const int seen = max(dense_length(A, seq) - (A.q_len - 1 - t), 1);
      for (int s = 0; s < splits; ++s) {
        if (!__syncthreads_or(!(fabsf(p[s * D + c]) < INFINITY))) continue;
        const int2 keys = A.keys[seq * A.splits + s];
        dense_again<D, PAGED>(A, bh, seq, div_group(h, A.Hq / Hkv), keys.x, min(keys.y, seen), p + s * D, ml + s);
      }
      __syncthreads();
      combine();
    }
  }
  if (half == 0) {
    A.out_o[bh * D + c] = (a + s_a[c]) / l;
    if (c == 0 && A.out_lse) A.out_lse[bh] = mall + logf(l);
  }
}

template <int D, bool PAGED, bool AGAIN>
hipError_t launch_dense_merge(const Plan& pl, DenseArgs& A, hipStream_t st) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dense_merge_kernel<D, PAGED, AGAIN>), dim3(pl.p.n_q_heads, pl.vbatch), dim3(2 * D), 0, st, A, pl.p.n_kv_heads);
  return hipGetLastError();
}

template <int D, bool PAGED>
hipError_t launch_dense_p(const Plan& pl, DenseArgs& A, hipStream_t st) {
  const vatt_params& p = pl.p;
  const int vectors = pl.q_len * pl.group, waves = dense_vector_waves(vectors);
  A.rounds = dense_rounds(vectors);
  if (dense_dots(pl.q_len, pl.group)) {
    dim3 grid(p.n_kv_heads, A.splits, p.batch);
    if (pl.group == 1) hipLaunchKernelGGL((dense_dot_kernel<D, 1, PAGED>), grid, dim3(kDenseThreads), 0, st, A);
    else hipLaunchKernelGGL((dense_dot_kernel<D, 2, PAGED>), grid, dim3(kDenseThreads), 0, st, A);
    return launch_dense_merge<D, false, false>(pl, A, st);
  }
  dim3 grid(p.n_kv_heads, (A.share ? A.share + p.batch : A.splits) * A.rounds, A.share ? 1 : p.batch);
  if (vectors <= 16) hipLaunchKernelGGL((dense_kernel<D, PAGED, 1, 1>), grid, dim3(kDenseThreads), 0, st, A);
  else if (waves == 1) hipLaunchKernelGGL((dense_kernel<D, PAGED, 2, 1>), grid, dim3(kDenseThreads), 0, st, A);
  else if (waves == 2) hipLaunchKernelGGL((dense_kernel<D, PAGED, 2, 2>), grid, dim3(kDenseThreads), 0, st, A);
  else hipLaunchKernelGGL((dense_kernel<D, PAGED, 2, 4>), grid, dim3(kDenseThreads), 0, st, A);
  return launch_dense_merge<D, PAGED, true>(pl, A, st);
}

template <int D>
hipError_t launch_dense_d(const Plan& pl, DenseArgs& A, hipStream_t st) {
  return pl.p.kv_layout == VATT_LAYOUT_PAGED ? launch_dense_p<D, true>(pl, A, st) : launch_dense_p<D, false>(pl, A, st);
}

// One workgroup per sequence: all threads read the current length, then copy the new K and V rows of
// every KV head (16 bytes per thread), then one thread stores length + 1.
template <bool PAGED>
__global__ void append_kernel(const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, uint16_t* k,
                              uint16_t* v, KVLayout L, int32_t* seq_lens, int n_max, int Hkv) {
  const int b = blockIdx.x;
  const int n = seq_lens[b];
  __syncthreads();
  if (n < 0 || n >= n_max) return;
  const int d = L.head_dim;
  const int per_head = d / 8;
  for (int t = threadIdx.x; t < Hkv * per_head; t += blockDim.x) {
    const int kvh = t / per_head, c = t % per_head;
    const int64_t src = ((int64_t)b * Hkv + kvh) * d + c * 8;
    const int64_t dst = kv_row_offset<PAGED>(L, b, kvh, n) + c * 8;
    *reinterpret_cast<uint4*>(k + dst) = *reinterpret_cast<const uint4*>(k_new + src);
    *reinterpret_cast<uint4*>(v + dst) = *reinterpret_cast<const uint4*>(v_new + src);
  }
  if (threadIdx.x == 0) seq_lens[b] = n + 1;
}

}  // namespace

hipError_t launch_dense(const Plan& pl, const void* q, const void* k, const void* v, const int32_t* block_table,
                        const int32_t* seq_lens, void* ws, float* out_o, float* out_lse, hipStream_t st) {
  DenseArgs A;
  A.q = static_cast<const uint16_t*>(q);
  A.k = static_cast<const uint16_t*>(k);
  A.v = static_cast<const uint16_t*>(v);
  A.Lk = pl.kv_k;
  A.Lk.block_table = block_table;
  A.Lv = pl.kv_v;
  A.Lv.block_table = block_table;
  A.seq_lens = seq_lens;
  A.part = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_dense_part);
  A.part_ml = reinterpret_cast<float2*>(A.part + (int64_t)pl.vbatch * pl.p.n_q_heads * pl.dense_splits * pl.p.head_dim);
  A.keys = reinterpret_cast<int2*>(A.part_ml + (int64_t)pl.vbatch * pl.p.n_q_heads * pl.dense_splits);
  A.out_o = out_o;
  A.out_lse = out_lse;
  A.batch = pl.p.batch;
  A.n_max = pl.p.n_max;
  A.Hq = pl.p.n_q_heads;
  A.splits = pl.dense_splits;
  A.share = pl.dense_share;
  A.q_len = pl.q_len;
  A.sm_scale = pl.sm_scale;
  if (pl.p.head_dim == 128) return launch_dense_d<128>(pl, A, st);
  if (pl.p.head_dim == 64) return launch_dense_d<64>(pl, A, st);
  return hipErrorInvalidValue;
}

hipError_t launch_append(const Plan& pl, const void* k_new, const void* v_new, void* k, void* v,
                         const int32_t* block_table, int32_t* seq_lens, hipStream_t st) {
  KVLayout L = pl.kv_k;
  L.block_table = block_table;
  const int threads = 128;
  if (pl.p.kv_layout == VATT_LAYOUT_PAGED)
    hipLaunchKernelGGL((append_kernel<true>), dim3(pl.p.batch), dim3(threads), 0, st,
                       static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new),
                       static_cast<uint16_t*>(k), static_cast<uint16_t*>(v), L, seq_lens, pl.p.n_max,
                       pl.p.n_kv_heads);
  else
    hipLaunchKernelGGL((append_kernel<false>), dim3(pl.p.batch), dim3(threads), 0, st,
                       static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new),
                       static_cast<uint16_t*>(k), static_cast<uint16_t*>(v), L, seq_lens, pl.p.n_max,
                       pl.p.n_kv_heads);
  return hipGetLastError();
}

}  // namespace vatt
