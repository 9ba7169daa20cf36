// Building blocks of the scoring kernels: the MFMA tile s = K_tile . Q^T of one wave, the staging
// of the query window in LDS, and the cross-lane sum over the queries of a token.
// (Alg. 1 step 1: "aggregate usage of each cached position from the last W queries".)
#ifndef AMS_SCORE_TILE_H
#define AMS_SCORE_TILE_H

#include <type_traits>

#include "ams_internal.h"

namespace ams {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

static constexpr float kNegInit = -3.0e38f;  // finite "minus infinity" for running maxima
static constexpr int kThreads = 256;

// MODE_LAST_LANES: last query, windows of 1, 2, 4, .. 32 queries.  The newest queries of all column blocks then sit in the same
// lanes, and a share in the score is the window's length times one in u, a power of two: the shares carry the score's weight
// 1 / (G Z), the score is what these lanes hold of the sum, and u is the sum over the length.  The bits of a sum of its own, without
// a multiply-add per logit and 16 registers; u keeps more where a share lies below 2^-126.  (With u's weight the score would lose up
// to five bits there.)  us per step with the sum and without: 152.4 and 149.5 (192 ragged units of up to 9001, 112 queries, 64 channels), 256.3 and 251.3 (25 of 44127, 224
// queries), 256.6 and 252.7 (276 of up to 5547 in one launch), 36.2 and 35.0 (32 of 1715); 8 others 0.99 to 1.01.
enum { MODE_MEAN = 0, MODE_LAST = 1, MODE_EXPECTED = 2, MODE_LAST_LANES = 3 };
inline bool newest_share_lanes(int window) { return window <= 32 && (window & (window - 1)) == 0; }

// Tiles of the one-launch scorer of which a CU holds two workgroups, four waves to a SIMD: at most 128 registers.  All but one take
// no more by themselves; the last-query score of 128 channels with a sum of its own took 129 to 132 and ran one workgroup on a CU:
// us per step 278.8 and 269.6 (500 units of 2000, a window of 24 queries), 355 and 339 (600), 547 and 524 (1000), 664 and 627 (1500
// of 1500); with the quotas in launches of their own 844 and 826 (2000 of 1500), 839 and 812 (3000 of 1000).
constexpr bool unit_tile_small(bool bf16, int nb, int head_dim) { return bf16 && nb <= (head_dim == 64 ? 2 : 1); }

struct ScoreArgs {
  KvDev k;
  Dims d;
  const int32_t* seq_lens;
  const char* q;
  float2* part;  // [units][n_chunks + 1][n_pad]  (max, sum) in the log2 domain; the last entry of a
                 // unit takes the tail blocks of a causal window
  float4* fin;   // [units][n_pad]  (M, weight for u, weight for g, query is real)
  float* u;
  float* g;
  int n_chunks, n_pad;
  int chunk;         // tokens per workgroup: a multiple of kMinScoreChunk, at most kScoreChunk
  float c2;          // log2(e) / sqrt(D)
  float inv_sqrt_d;  // 1 / sqrt(D)
  // optional by-products for Eq. (1) and the EMA (NULL: not wanted): per chunk the sum of
  // max(u,0)+eps from the second sweep; the unit's sum of the credit before the update, formed by the
  // kernel that merges the statistics and carried in the first chunk's entry
  double2* vc_part;     // [units][n_chunks]
  const float* credit;  // [units][t_stride]
  double* csum;         // [units]
  double* ksum;         // [units][n_chunks][D]: sums of the keys (or of the unit vectors); NULL: nobody wants them here
  double2* soft;        // [units][n_chunks]: (max, sum of exp) of the scores in g, left by the sweep that forms them; may be NULL
  float eps;
  bool even;    // the n_chunks chunks of a unit share the cache evenly, whatever its length up to t_max
  bool compact; // ragged batch: the workgroups of the sweeps count only the chunks that exist
  bool fold;    // the second sweep merges the first one's statistics itself (no reduction kernel between them)
  bool causal;  // causal window (App. A): query w of the window sees keys 0 .. T-W+w
  int32_t* status;  // word the one-read scorer raises when a bounded wait expires; the two-sweep path clears it
};

// Raises a kernel's dynamic LDS limit once per kernel and device (not before every launch).
template <auto Kernel>
inline hipError_t ensure_lds(int bytes) {
  constexpr int kMaxDevices = 64;
  static int granted[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (granted[dev] >= bytes) return hipSuccess;
  e = hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) granted[dev] = bytes;
  return e;
}

// Tokens per chunk of a cache of T positions (at t_max a.chunk either way, without the division's 0.2 us in front of the keys).
__device__ __forceinline__ int chunk_len(const ScoreArgs& a, int T) {
  return a.even && T != a.d.t_max ? even_chunk(T, a.n_chunks) : a.chunk;
}

// Row geometry of a cache of HD channels: bytes per row, stride of a query row in LDS (bf16, or the three bf16 terms of an
// fp32 row one behind the other; padded by 16 bytes against bank conflicts), 16-byte vectors per half row (what one lane
// feeds the MFMA).
template <bool BF16, int HD = 128>
struct Tr {
  static_assert(HD == 64 || HD == 128, "head dimensions the tiles are written for");
  static constexpr int kRowBytes = HD * (BF16 ? 2 : 4), kAVecs = kRowBytes / 32;
  static constexpr int kQTerm = HD * 2, kQStride = kQTerm * (BF16 ? 1 : 3) + 16;
};

// fp32 values as sums of three bf16 terms, each the rest rounded to nearest: 24 bits hold exactly.  A value that is no
// number, infinite or rounds to infinity has SAFE's terms: itself (truncated) alone.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t round2_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, bf16x2));
}
__device__ __forceinline__ bool infinite_or_nan(uint32_t bits) { return (bits & 0x7F800000u) == 0x7F800000u; }
template <bool SAFE>
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = round2_bf16(a, b);
  if (SAFE) {
    if (infinite_or_nan(hi << 16)) hi = (hi & 0xFFFF0000u) | (__float_as_uint(a) >> 16);
    if (infinite_or_nan(hi)) hi = (hi & 0xFFFFu) | (__float_as_uint(b) & 0xFFFF0000u);
  }
  float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xFFFF0000u);
  if (SAFE) {  // (not for a NaN, whose first term may have come out as an infinity: its rest is a NaN)
    if (fabsf(a) == INFINITY) ra = 0.f;
    if (fabsf(b) == INFINITY) rb = 0.f;
  }
  mid = round2_bf16(ra, rb);
  lo = round2_bf16(ra - __uint_as_float(mid << 16), rb - __uint_as_float(mid & 0xFFFF0000u));
}

// Makes the keys opaque where they are, so that terms formed from them before are formed again instead of being kept.
template <int N>
__device__ __forceinline__ void forget_terms(const uint4 (&av)[N]) {
  auto& v = const_cast<uint4(&)[N]>(av);
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i].x), "+v"(v[i].y), "+v"(v[i].z), "+v"(v[i].w));
}

// 16 bytes (column col) of a query row -> its place in LDS; fp32: times 2^-exp, and the largest magnitude -> top.
template <bool BF16, int HD>
__device__ __forceinline__ void store_q(char* row, int col, const uint4& v, float& top, int exp = 0) {
  if constexpr (BF16) {
    *(uint4*)(row + col * 16) = v;
  } else {
    float4 x = __builtin_bit_cast(float4, v);
    top = fmaxf(fmaxf(top, fmaxf(fabsf(x.x), fabsf(x.y))), fmaxf(fabsf(x.z), fabsf(x.w)));
    if (exp != 0) x = make_float4(ldexpf(x.x, -exp), ldexpf(x.y, -exp), ldexpf(x.z, -exp), ldexpf(x.w, -exp));
    uint2 t[3];
    split2<true>(x.x, x.y, t[0].x, t[1].x, t[2].x);
    split2<true>(x.z, x.w, t[0].y, t[1].y, t[2].y);
#pragma unroll
    for (int j = 0; j < 3; ++j) *(uint2*)(row + j * Tr<BF16, HD>::kQTerm + col * 8) = t[j];
  }
}

// Query window of the unit -> LDS, rows padded against bank conflicts, rows >= N zero.  Returns the largest magnitude that the
// thread has seen (fp32).
template <bool BF16, int NB, int HD = 128, int THREADS = kThreads>
__device__ __forceinline__ float load_q(const ScoreArgs& a, int l, int b, int h, char* qlds, int exp = 0) {
  constexpr int RB = Tr<BF16, HD>::kRowBytes, QS = Tr<BF16, HD>::kQStride, CPR = RB / 16;
  const char* src = a.q + ((((int64_t)l * a.d.B + b) * a.d.H + h) * a.d.G) * (int64_t)a.d.W * RB;
  float top = 0.f;
  for (int ch = threadIdx.x; ch < NB * 32 * CPR; ch += THREADS) {
    const int n = ch / CPR, col = ch % CPR;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < a.d.N) v = *(const uint4*)(src + (int64_t)n * RB + col * 16);
    store_q<BF16, HD>(qlds + n * QS, col, v, top, exp);
  }
  return top;
}

// Barrier after load_q.  fp32: bf16 terms are cut short below 2^-109 (the last one ends at 2^-133), which shows where the
// other factor is about as large: keys of 2^-118 against queries of 2^118 had logits off by 1e-5.  A window whose largest
// entry lies outside 2^-100 .. 2^100 is loaded again, scaled to about one, and the power of two taken from it, which is
// returned (0 otherwise), goes to the keys (tile_mma).  An ordinary window waits for one more read of LDS: 37.2 -> 37.6 to 37.9
// us per step for 8 units of 4096 positions, no difference in launches of 100 us and more.
template <bool BF16, int NB, int HD = 128, int THREADS = kThreads>
__device__ __forceinline__ int settle_q(const ScoreArgs& a, int l, int b, int h, char* qlds, float top) {
  if constexpr (BF16) {
    __syncthreads();
    return 0;
  } else {
    constexpr int WAVES = THREADS / 64;
    __shared__ __align__(16) int seen[WAVES];
    __shared__ float tops[WAVES];
    seen[threadIdx.x >> 6] = (__any(top >= 0x1p-100f) ? 1 : 0) | (__any(top >= 0x1p100f) ? 2 : 0);
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; w += 4) {
      const int4 s4 = *(const int4*)&seen[w];
      all |= (s4.x | s4.y) | (s4.z | s4.w);
    }
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(all) == 1, 1)) return 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    tops[threadIdx.x >> 6] = top;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) top = fmaxf(top, tops[w]);
    if (!(top > 0.f) || top == INFINITY) return 0;
    const int exp = __builtin_amdgcn_readfirstlane(max(-126, min(126, __builtin_amdgcn_frexp_expf(top) - 1)));
    load_q<BF16, NB, HD, THREADS>(a, l, b, h, qlds, exp);
    __syncthreads();
    return exp;
  }
}

// Lane (r = lane % 32, hf = lane / 32) reads the hf-th half of row t0 + r: one contiguous piece
// (128 bytes for bf16 rows of 128 channels).  The contraction index is permuted the same way on
// the query side, which leaves the dot products unchanged.
template <bool BF16, int HD = 128>
__device__ __forceinline__ void load_a(const ScoreArgs& a, int l, int b, int h, int t0, int T,
                                       int lane, uint4 (&av)[Tr<BF16, HD>::kAVecs],
                                       const int32_t* blk_lds = nullptr, int blk_t0 = 0) {
  constexpr int NV = Tr<BF16, HD>::kAVecs;
  // rows past the end re-read the last row (no divergent branch); their logits are masked later
  const int t = min(t0 + (lane & 31), T - 1);
  const char* row;
  if (blk_lds) {
    // paged cache: the physical block numbers of the positions from blk_t0 (a multiple of 16) on
    // were staged in LDS, so the row address does not wait for a table entry from memory
    int64_t slot = (int64_t)blk_lds[(t - blk_t0) >> 4] * 16 + (t & 15);
    slot = slot < 0 ? 0 : (slot >= a.k.n_slots ? a.k.n_slots - 1 : slot);
    row = a.k.base + (((int64_t)l * a.k.n_slots + slot) * a.k.H + h) * (int64_t)a.k.row_bytes;
  } else {
    row = kv_row(a.k, l, b, h, t);
  }
  const uint4* p = (const uint4*)(row + (lane >> 5) * (Tr<BF16, HD>::kRowBytes / 2));
#pragma unroll
  for (int i = 0; i < NV; ++i) av[i] = p[i];
}

// Paged cache: block numbers of the positions [c0, t_lim) of sequence b -> LDS (c0 a multiple of 16).
template <int THREADS = kThreads>
__device__ __forceinline__ void stage_blocks(const ScoreArgs& a, int b, int c0, int t_lim, int32_t* blk_lds) {
  const int n = (t_lim - c0 + 15) >> 4;
  for (int i = threadIdx.x; i < n; i += THREADS)
    blk_lds[i] = a.k.block_table[(int64_t)b * a.k.max_blocks + (c0 >> 4) + i];
  __syncthreads();
}

// fp32 tile by bf16 matrix instructions: with K = K1 + K2 + K3 and Q = Q1 + Q2 + Q3 (bf16 terms, each 2^-9 of the one before)
// the six products down to 2^-18 are kept, K3 Q1 + K1 Q3 + K2 Q2 + K2 Q1 + K1 Q2 + K1 Q1; what is left out is 2^-26 of a
// product.  One v_mfma_f32_32x32x16_bf16 takes half the time of a v_mfma_f32_32x32x2_f32 and does eight times its work, so
// that six of them cost 3/8; the terms of K take 5.5 vector instructions per value.  Products are exact and 16 of them are
// added per step, where the fp32 instruction rounds after two: against 64 bits the usage is off by 1.9e-7 (2-norm, 8 units of
// 4096 positions), 2.4e-7 with the fp32 instruction.  us per step, with it and with this: 408 and 290 (20 units of 30000, 128
// queries), 419 and 239 (130 of 3000), 238 and 194 (20 of 30000, 64 queries), 175 and 165 (8 queries: memory bound), 240 and
// 170 (176 ragged units of up to 2772, 64 queries).
// SAFE: keys that are infinite or no number (K1 holds them, and the products with Q2 and Q3, which may be zero, leave them out),
// and keys that take a power of two from the queries (settle_q).
template <int NB, int HD, bool SAFE, bool AHEAD>
__device__ __forceinline__ void tile_split(const uint4 (&av)[Tr<false, HD>::kAVecs], const char* qb, floatx16 (&acc)[NB], int key_exp = 0) {
  constexpr int QS = Tr<false, HD>::kQStride, QT = Tr<false, HD>::kQTerm;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
  struct Terms {
    uint32_t h[4], m[4], l[4], f[4];  // K1, K2, K3, and K1 without what is infinite or no number
  };
  auto split = [&](int ks) __attribute__((always_inline)) {
    float4 x0 = __builtin_bit_cast(float4, av[2 * ks]), x1 = __builtin_bit_cast(float4, av[2 * ks + 1]);
    if (SAFE) {
      x0 = make_float4(ldexpf(x0.x, key_exp), ldexpf(x0.y, key_exp), ldexpf(x0.z, key_exp), ldexpf(x0.w, key_exp));
      x1 = make_float4(ldexpf(x1.x, key_exp), ldexpf(x1.y, key_exp), ldexpf(x1.z, key_exp), ldexpf(x1.w, key_exp));
    }
    Terms t;
    split2<SAFE>(x0.x, x0.y, t.h[0], t.m[0], t.l[0]);
    split2<SAFE>(x0.z, x0.w, t.h[1], t.m[1], t.l[1]);
    split2<SAFE>(x1.x, x1.y, t.h[2], t.m[2], t.l[2]);
    split2<SAFE>(x1.z, x1.w, t.h[3], t.m[3], t.l[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t.f[i] = t.h[i];
      if (SAFE)
        t.f[i] = (infinite_or_nan(t.h[i] << 16) ? 0u : t.h[i] & 0xFFFFu) | (infinite_or_nan(t.h[i]) ? 0u : t.h[i] & 0xFFFF0000u);
    }
    return t;
  };
  auto frag = [](const uint32_t (&t)[4]) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, make_uint4(t[0], t[1], t[2], t[3]));
  };
  constexpr int NK = HD / 16, kBuf = AHEAD ? 2 : 1;  // AHEAD: the next step's terms are formed and read a step ahead
  Terms t[kBuf];
  uint4 q[kBuf][NB][3];
  auto fetch = [&](int ks) __attribute__((always_inline)) {
    t[ks % kBuf] = split(ks);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 3; ++j) q[ks % kBuf][nb][j] = *(const uint4*)(qb + nb * 32 * QS + ks * 16 + j * QT);
  };
  if (kBuf == 2) fetch(0);
#pragma unroll
  for (int ks = 0; ks < NK; ++ks) {
    if (kBuf == 1) fetch(ks);
    if (kBuf == 2 && ks + 1 < NK) fetch(ks + 1);
    const Terms& k = t[ks % kBuf];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const bf16x8 Q1 = __builtin_bit_cast(bf16x8, q[ks % kBuf][nb][0]), Q2 = __builtin_bit_cast(bf16x8, q[ks % kBuf][nb][1]),
                   Q3 = __builtin_bit_cast(bf16x8, q[ks % kBuf][nb][2]);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.l), Q1, acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.f), Q3, acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.m), Q2, acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.m), Q1, acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.f), Q2, acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(k.h), Q1, acc[nb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);  // a step's terms at a time: hoisted further, they do not fit the registers
  }
}

// acc[nb][i] = s_raw[token 8*(i/4) + 4*hf + i%4][query nb*32 + lane%32]
// (CLEAR = false: acc starts from what it holds; AHEAD: registers to spare, see tile_split)
template <bool BF16, int NB, int HD = 128, bool CLEAR = true, bool AHEAD = true>
__device__ __forceinline__ void tile_mma(const uint4 (&av)[Tr<BF16, HD>::kAVecs], const char* qlds,
                                         int lane, floatx16 (&acc)[NB], int key_exp = 0) {
  constexpr int QS = Tr<BF16, HD>::kQStride;
  [[maybe_unused]] constexpr int NV = Tr<BF16, HD>::kAVecs;
  const char* qb = qlds + (lane & 31) * QS + (lane >> 5) * (Tr<BF16, HD>::kQTerm / 2);
  if constexpr (BF16) {
#pragma unroll
    for (int nb = 0; nb < NB && CLEAR; ++nb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NV; ++ks) {
      const bf16x8 A = __builtin_bit_cast(bf16x8, av[ks]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const uint4 bv = *(const uint4*)(qb + nb * 32 * QS + ks * 16);
        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, bv), acc[nb], 0, 0, 0);
      }
    }
  } else {
    tile_split<NB, HD, false, AHEAD && NB <= 2>(av, qb, acc);
    float t = 0.f;  // a key that is infinite or no number shows in every column
#pragma unroll
    for (int i = 0; i < 16; ++i) t = __builtin_fmaf(acc[0][i], 0.f, t);
    if (__builtin_expect(__any(t != 0.f) || key_exp != 0, 0)) {
      forget_terms(av);
      int off = 0;
      asm volatile("" : "+s"(off));
      tile_split<NB, HD, true, false>(av, qb + off, acc, key_exp);
    }
  }
}

__device__ __forceinline__ int acc_row(int i, int hf) { return 8 * (i >> 2) + 4 * hf + (i & 3); }

// Software pipeline over the column blocks of a tile (bf16 caches): the query fragments of a column
// block are read from LDS a whole column block before the matrix instructions that use them, and the
// matrix instructions of column block nb + 1 are issued between the vector instructions that consume
// column block nb.  A wave then neither waits for LDS in front of every MFMA nor leaves one of the
// two pipes idle while it uses the other.
//   col_frags   this lane's 16-byte query fragments of one column block -> registers
//   col_mma     acc = K_block . Q_col^T from fragments in registers
//   col_hints   scheduling hints for one step of the pipeline (STEPS matrix instructions, each
//               followed by VALU_PER vector and TRANS_PER transcendental instructions)
template <bool BF16, int HD = 128>
__device__ __forceinline__ void col_frags(const char* qb, uint4 (&bq)[Tr<BF16, HD>::kAVecs]) {
#pragma unroll
  for (int ks = 0; ks < Tr<BF16, HD>::kAVecs; ++ks) bq[ks] = *(const uint4*)(qb + ks * 16);
}
template <bool BF16, int HD = 128, bool CLEAR = true>
__device__ __forceinline__ void col_mma(const uint4 (&av)[Tr<BF16, HD>::kAVecs],
                                        const uint4 (&bq)[Tr<BF16, HD>::kAVecs], floatx16& acc) {
  static_assert(BF16, "the pipelined walk is written for bf16 caches");
#pragma unroll
  for (int i = 0; i < 16 && CLEAR; ++i) acc[i] = 0.f;
#pragma unroll
  for (int ks = 0; ks < Tr<BF16, HD>::kAVecs; ++ks)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[ks]), __builtin_bit_cast(bf16x8, bq[ks]),
                                                  acc, 0, 0, 0);
}
template <int STEPS, int VALU_PER, int TRANS_PER, bool READS>
__device__ __forceinline__ void col_hints() {
  if (READS) __builtin_amdgcn_sched_group_barrier(0x100, STEPS, 0);  // the LDS reads of the column block after next, first
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);         // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER, 0);  // vector ALU
    if (TRANS_PER > 0) __builtin_amdgcn_sched_group_barrier(0x400, TRANS_PER, 0);  // exp2
  }
}

// Sum (or maximum) of 16 per-lane values over the 32 lanes of a half wave, halving the number of live values
// at every exchange.  Lane c ends up with the total of value index c >> 1.
// Exchanges: rows of 16 lanes swap through v_permlane16_swap (bit 4 of the lane), then DPP
// row_ror:8 (bit 3), row_half_mirror (lane <-> 7 - lane inside groups of 8: the partner has the
// opposite bit 2), quad_perm xor 2 (bit 1) and xor 1; no LDS traffic.
__device__ __forceinline__ float dpp_ror8(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_half_mirror(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x141, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_xor2(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x4E, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_xor1(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0xB1, 0xf, 0xf, true));
}
template <bool MAX = false>
__device__ __forceinline__ float reduce16_over32(const float (&v)[16], int c) {
  auto op = [](float x, float y) __attribute__((always_inline)) { return MAX ? fmaxf(x, y) : x + y; };
  float w8[8], w4[4], w2[2];
  const bool b3 = c & 8, b2 = c & 4, b1 = c & 2;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // even rows receive the partner row's v[j], odd rows the partner row's v[j + 8]
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 8]), false, false);
    w8[j] = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float keep = b3 ? w8[j + 4] : w8[j], send = b3 ? w8[j] : w8[j + 4];
    w4[j] = op(keep, dpp_ror8(send));
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float keep = b2 ? w4[j + 2] : w4[j], send = b2 ? w4[j] : w4[j + 2];
    w2[j] = op(keep, dpp_half_mirror(send));
  }
  const float keep = b1 ? w2[1] : w2[0], send = b1 ? w2[0] : w2[1];
  const float w1 = op(keep, dpp_xor2(send));
  return op(w1, dpp_xor1(w1));
}

// The last-query score of token c >> 1 from the sums of all queries (MODE_LAST_LANES).
__device__ __forceinline__ float newest_lanes(const float (&pu)[16], int c, int window) {
  float v[16];
  const bool newest = (c & (window - 1)) == window - 1;
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = newest ? pu[i] : 0.f;
  return reduce16_over32(v, c);
}

}  // namespace ams
#endif
