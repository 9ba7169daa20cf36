// The two sweeps over K and the reduction between them (see score.hip for the method): kernels and launchers, shared by
// the plain scorers (score.hip) and the scorers that need the keys themselves as well (score_keys.hip).
#ifndef AMS_SCORE_SWEEP_H
#define AMS_SCORE_SWEEP_H

#include <type_traits>

#include "score_tile.h"
#include "sweep_grid.h"

namespace ams {
namespace {

// ---------------------------------------------------------------------------------------------
// Both sweeps walk a chunk of tokens (kMinScoreChunk .. kScoreChunk, chosen on the host so that short caches
// still give the chip enough workgroups) in 32-token blocks per wave.  The keys of the next block are
// requested before the current block is multiplied (two register buffers, used alternately), and
// the query columns are processed in groups of kGroup<NB> blocks of 32 so that only that many
// accumulator tiles are live at a time: more bytes in flight per wave at the same occupancy.
// ---------------------------------------------------------------------------------------------
#ifndef AMS_SCORE_GROUP_DIV
#define AMS_SCORE_GROUP_DIV 2   // column blocks of a wave are processed in this many groups (tuning knob)
#endif
#ifndef AMS_SCORE_MIN_WAVES
#define AMS_SCORE_MIN_WAVES 3   // waves per SIMD the register allocation aims for (tuning knob)
#endif
template <int NB>
constexpr int kGroup = (NB % AMS_SCORE_GROUP_DIV == 0 && NB >= 4) ? NB / AMS_SCORE_GROUP_DIV : NB;
// With five or more column blocks (bf16 caches, plain sweeps; two waves per SIMD either way) a block is
// walked as a software pipeline over its column blocks (score_tile.h: col_frags / col_mma / col_hints):
// two accumulator tiles and two sets of query fragments live instead of all accumulator tiles, the
// matrix cores and the vector ALU busy together for longer (30 % of the cycles against 17 %).  Measured
// at 224 queries per key, same machine: 1.064 + 0.938 ms for the two sweeps against 1.095 + 0.978.  With
// four column blocks it does not pay: three waves per SIMD do not fit the extra registers (and spill),
// and the two-wave moment-sum kernel is unchanged by it (0.617 ms either way).
#ifndef AMS_SCORE_PIPE_MIN_NB
#define AMS_SCORE_PIPE_MIN_NB 5
#endif
// Column blocks without padding, whatever the number of queries that NB column blocks are taken for (NB of 1, 2, 4, 7, 8).
template <int NB>
constexpr int kFullBlocks = NB == 8 ? 7 : NB == 7 ? 4 : NB / 2;
template <bool BF16, int NB, bool TAIL>
constexpr bool kPipe = BF16 && !TAIL && NB >= AMS_SCORE_PIPE_MIN_NB;

// (maximum, sum of exp relative to it) of n scores -> *out, in double, by the whole workgroup; lanes, then waves,
// combined in a fixed order.  An empty partial is (-inf, 0).
template <int THREADS = kThreads>
__device__ __forceinline__ void softmax_part(const float* e, int n, double2* out) {
  __shared__ double2 sm[THREADS / 64];
  float mf = -INFINITY;
  for (int t = threadIdx.x; t < n; t += THREADS) mf = fmaxf(mf, e[t]);
  double m = (double)mf, z = 0.0;
  if (mf != -INFINITY)
    for (int t = threadIdx.x; t < n; t += THREADS) z += exp((double)e[t] - m);
  auto merge = [](double& m1, double& z1, double m2, double z2) __attribute__((always_inline)) {
    const double mx = fmax(m1, m2);
    if (mx == -INFINITY) return;
    z1 = z1 * exp(m1 - mx) + z2 * exp(m2 - mx);
    m1 = mx;
  };
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double m2 = __shfl_xor(m, o), z2 = __shfl_xor(z, o);
    // both partners must arrive at the same value: combine in lane order
    double ml = (threadIdx.x & o) ? m2 : m, zl = (threadIdx.x & o) ? z2 : z;
    const double mh = (threadIdx.x & o) ? m : m2, zh = (threadIdx.x & o) ? z : z2;
    merge(ml, zl, mh, zh);
    m = ml;
    z = zl;
  }
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = make_double2(m, z);
  __syncthreads();
  if (threadIdx.x == 0) {
    double M = sm[0].x, Z = sm[0].y;
    for (int w = 1; w < THREADS / 64; ++w) merge(M, Z, sm[w].x, sm[w].y);
    *out = make_double2(M, Z);
  }
}

// What a sweep does with the keys besides the products with the queries.
enum { KEYS_NONE = 0, KEYS_MEAN = 1, KEYS_COS = 2 };
// Moment sums of the first sweep: none, of the logits relative to the first query's, of the centred logits.
enum { MOMENTS_NONE = 0, MOMENTS_FIRST = 1, MOMENTS_CENTRED = 2 };

// Squared lengths of a block's keys: K . K^T on the matrix cores, of which the diagonal is wanted.  Token r sits in lane
// r of the half wave (r >> 2) & 1, in register 4 * (r >> 3) + (r & 3).
template <int HD>
__device__ __forceinline__ floatx16 key_gram(const uint4 (&av)[Tr<true, HD>::kAVecs]) {
  floatx16 acc;
  col_mma<true, HD>(av, av, acc);
  return acc;
}

// The squared length of token c, valid in the lane of its half wave that holds it.
__device__ __forceinline__ float key_norm2(const floatx16& gram, int c) {
  float n2 = gram[0];
  const int own = 4 * (c >> 3) + (c & 3);
#pragma unroll
  for (int i = 1; i < 16; ++i) n2 = own == i ? gram[i] : n2;
  return n2;
}

// Adds a block's keys to this lane's running sums.  A key tile times the identity is the tile itself with one channel per
// lane and 16 tokens in its registers (exact), which are then added up in double like in the streaming kernels: keys that
// cancel leave a sum far below their size.  ident: the two halves of the identity, one per 8 columns.
template <int HD, bool COS>
__device__ __forceinline__ void add_keys(const uint4 (&av)[Tr<true, HD>::kAVecs], const uint4 (*ident)[64], double* inv_len,
                                         int lane, int rows, double (&sum)[HD / 32]) {
  const int hf = lane >> 5;
  if (COS) {  // 1 / length of the block's tokens (0 for a zero key and for rows past the end), through LDS
    const int c = lane & 31;
    const float n2 = key_norm2(key_gram<HD>(av), c);
    if (((c >> 2) & 1) == hf) inv_len[c] = (n2 > 0.f && c < rows) ? rsqrt((double)n2) : 0.0;
    // the wave's own LDS accesses stay in order; the compiler must keep them so
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  int off = 0;
  asm volatile("" : "+s"(off));  // the identity is re-read per block: registers are scarcer than LDS reads
  const bf16x8 I0 = __builtin_bit_cast(bf16x8, ident[0][lane + off]), I1 = __builtin_bit_cast(bf16x8, ident[1][lane + off]);
#pragma unroll
  for (int cb = 0; cb < HD / 32; ++cb) {
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[2 * cb]), I0, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[2 * cb + 1]), I1, acc, 0, 0, 0);
    double t[2] = {sum[cb], 0.0};  // two independent chains
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (COS)
        t[i & 1] = __builtin_fma((double)acc[i], inv_len[acc_row(i, hf) + off], t[i & 1]);
      else
        t[i & 1] += acc_row(i, hf) < rows ? (double)acc[i] : 0.0;
    }
    sum[cb] = t[0] + t[1];
  }
}
// Channel whose sum lane n of a half wave holds in sum[cb].
template <int HD>
__device__ __forceinline__ int key_channel(int cb, int n) {
  return (n >> 4) * (HD / 2) + cb * 16 + (n & 15);
}

// Threads of a sweep workgroup: eight waves where the query window leaves room for one workgroup on a CU only.
template <bool BF16, int NB, int HD>
constexpr int kSweepThreads = !BF16 && NB == 4 && HD == 128 ? 2 * kThreads : kThreads;

// ---------------------------------------------------------------------------------------------
// Sweep 1: per chunk, per query (max, sum exp2) of the scaled logits.
// ---------------------------------------------------------------------------------------------
//
// Causal window (App. A "Mass construction"): query w of the window sits at position T-W+w and sees
// the keys up to its own position.  The 32-token blocks that lie entirely before the newest W-1 keys
// are seen by every query and run like those of the plain sweeps, which then stop at t_end; the few
// blocks from t_end on go to one workgroup more per unit, the last ones of the launch, where a (query, key) pair
// the mask hides is left out.  As launches of their own they took 7 to 16 us each; beside the others they cost nothing in
// large launches and 1 to 4 us in small ones: us per step 106 and 91 (64 units of 4000), 252 and 229 (40 of 30000, 224 queries), 65
// and 52 (6 of 1090 with the paper's options, without the reduction's launch as well), 1055 and 1044 (256 of 32768, no further apart
// than the runs of one side).  Mixed
// in with the units' chunks (one of them first in every unit) they break the order of the key stream: 1092, 99, 241; 100 units
// of 20000 take 320 in two launches, 362 mixed and 298 at the end.
//
// Which (unit, chunk) a workgroup of the sweeps takes.  Dense caches: grid x = chunk, grid y = unit.
// Paged caches keep the rows of a position's KV heads next to each other in a slot, so there the
// heads of one (layer, sequence, chunk) are given to consecutive workgroups: they run at the same
// time and read the same slots (DRAM pages) together instead of eight separate times.  Consecutive workgroups go to
// consecutive XCDs, so without more each XCD would read one head, the same 256 of every 2048 bytes, all through the
// launch; the heads therefore move on by one every eighth (layer, sequence, chunk).  4096 ragged units, 8 heads: 6025 us
// per step against 6447; moving on every time, or every second time, gives 6490 and 6267, every 16th or 64th 6007 to 6008.
// 4 heads gain as well (2048 units, 3396 -> 3080); with 1, 2 or 3 heads, or rows of 128 bytes, it makes no difference (3537
// and 3571, 3727 and 3700, 2333 and 2344; 3581 and 3559 for 8 heads).
//
// Ragged batches (compact): the chunks past the end of a sequence are left out of the count, so that the workgroups that have
// work are the first ones of the launch, without gaps.  With a grid of (chunk, unit) the gaps repeat with the batch and leave
// some XCDs more work than others: 192 units of 700 to 9001 positions 161 -> 145 us per step, 768 paged units of 2354 to 5384
// 560 -> 509, 4096 paged ones of 4096 to 16384 5655 -> 5557.  A sequence per lane, so at most 64 of them.
__device__ __forceinline__ int causal_t_end(const ScoreArgs& a, int T, bool causal) {
  return causal ? max(0, (T - a.d.W + 1) / 32 * 32) : T;
}
// Returns whether it is the unit's tail of a causal window.
template <bool CAUSAL>
__device__ __forceinline__ bool sweep_tile(const ScoreArgs& a, bool reversed, int& unit, int& chunk) {
  int bx = blockIdx.x, by = blockIdx.y;
  const int chunks = CAUSAL ? a.n_chunks : (int)gridDim.x;
  if constexpr (CAUSAL) {
    sweep_place(blockIdx.x, blockIdx.y, gridDim.x, chunks, bx, by);
    if (by >= a.d.units) {
      unit = sweep_tail(bx, by, chunks, a.d.units);
      chunk = unit < 0 ? -1 : 0;
      return true;
    }
  }
  if (a.compact) {
    const int lane = threadIdx.x & 63, B = a.d.B, H = a.d.H;
    const int len = lane < B ? max(0, min(a.seq_lens[lane], a.d.t_max)) : 0;
    const int n = (causal_t_end(a, len, CAUSAL) + a.chunk - 1) / a.chunk;  // chunks of this lane's sequence
    int incl = n;
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);  // row_shr: 1, 2, 4, 8
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);  // row_bcast: 15, 31
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);
    const int per_layer = __builtin_amdgcn_readlane(incl, 63), total = per_layer * H * a.d.L;
    int lin = by * chunks + bx;
    unit = 0;
    chunk = a.n_chunks;  // past every sequence: nothing to do
    if (lin >= total) return false;
    if (reversed) lin = total - 1 - lin;
    int rest, h = 0;  // (sequence, chunk) of the layer, counted over what there is
    int l;
    if (a.k.layout == AMS_LAYOUT_PAGED) {
      const int r = lin / H;
      h = (lin + r / 8) % H;
      l = r / per_layer;
      rest = r - l * per_layer;
    } else {
      l = lin / (per_layer * H);
      rest = lin - l * per_layer * H;
    }
    const int scale = a.k.layout == AMS_LAYOUT_PAGED ? 1 : H;
    const int b = __popcll(__ballot(lane < B && incl * scale <= rest));  // sequences that end before it
    const int nb = __builtin_amdgcn_readlane(n, b);
    rest -= (__builtin_amdgcn_readlane(incl, b) - nb) * scale;
    if (scale > 1) {
      h = rest / nb;
      rest -= h * nb;
    }
    chunk = rest;
    unit = (l * B + b) * H + h;
    return false;
  }
  if (reversed) {
    bx = chunks - 1 - bx;
    by = a.d.units - 1 - by;
  }
  if (a.k.layout != AMS_LAYOUT_PAGED) {
    unit = by;
    chunk = bx;
    return false;
  }
  const int lin = by * chunks + bx;
  const int rest = lin / a.d.H, h = (lin + rest / 8) % a.d.H;
  chunk = rest % chunks;
  unit = (rest / chunks) * a.d.H + h;
  return false;
}

// The reference of the exponentials follows the running maximum, so that the largest logit of a wave has the exponent 0.  A
// reference taken from the wave's first block alone saves the maxima (2239 -> 2167 us per step for 112 units of 131072
// positions, 224 queries), but a later, dominant key then has an exponent of up to 24 in fp32, which costs its share 1e-6;
// larger ones need the wave's blocks again, and the moment sweep next to it took 1949 us instead of 1858 (65536 positions).
//
// KEYS (key-diversity and redundancy-aware scores, bf16 caches): the sums of the keys, or of the unit vectors, that those
// scores need ride along with the first sweep, and their dot products with the keys along with the second, so that K is
// streamed twice and not four times (score_keys.hip).  The unit vectors take two waves per SIMD: with the registers of
// three the first sweep spills (1281 against 1415 us per step for 256 units of 32768 positions).  With seven or eight column
// blocks of 128 channels the pipeline over them spills at two waves as well (52 and 56 registers): there the blocks are taken
// in two groups of accumulator tiles (none and 13; 1894 -> 1451 us for 112 units of 65536 positions and 224 queries, 894 ->
// 791 for 256 units of 8192 and 256 queries, where the streaming kernels take 790).
//
// MOMENTS (expected-attention score, Sec. 3.3 plug-in scorer): the log of the Gaussian moment of the
// window's queries is mean_n s + var_n s / 2 over the N logits of a token.  It needs no softmax
// statistics, so it is formed here, where few registers are live.  Raw logits are used: the causal mask does not apply.
// Centred form (bf16): the mean logit of a token is its product with the mean query, which takes part as three bf16 terms
// that add up to its fp32 value, the same in all columns of a tile; the products with the queries then start from minus
// that tile, so that the accumulators are s - mean and the variance is one multiply-add per logit (24 more matrix
// instructions per block of 32 keys, one vector instruction per logit for the variance and one for s itself instead of four,
// one reduction over the lanes instead of three).  It gains with 64 channels (1 to 14 %; 454 -> 428 us per step for 256 units of
// 16384 positions) and with three or four column blocks of 128 in launches of 512 workgroups and more (1134 -> 1109 us for 256
// units of 32768, 335 -> 317 for 512 of 4096; 439 -> 450 for 304 of 9000, the worst of nine).  Its own start, two barriers,
// costs 1 us in smaller ones; with one or two column blocks of 128 channels the products are not hidden (319 -> 327 for 144
// units of 16589, 64 queries), and with seven or eight it spills (1835 -> 1933, 659 -> 958).  There, in the causal tail and for
// fp32 caches, and for a wave whose statistics come out as no numbers, the sums are those of (s - r) and (s - r)^2 with r the
// token's logit against the unit's first query (a reference close to the mean keeps the subtraction of the squares harmless).
template <bool BF16, int NB, int MOMENTS, int HD, int KEYS>
struct StatsLds {
  static constexpr int kWaves = kSweepThreads<BF16, NB, HD> / 64;
  static constexpr bool kCentred = MOMENTS == MOMENTS_CENTRED;
  __align__(16) char mean[kCentred ? 3 * HD * 2 : 16];  // minus the mean query in three bf16 terms
  __align__(16) float g[MOMENTS ? kScoreChunk : 4];     // the chunk's moment scores, written once at the end
  float2 xch[kCentred ? 1 : kWaves][NB * 32];
  int32_t blk[kScoreChunk / 16];  // paged caches: this chunk's block numbers
  int mean_cut;                   // the terms do not add up to the mean query
};

// XCH_IN_Q: the exchange takes the place of the query window (the centred sweep needs the room).
template <bool BF16, int NB, bool CAUSAL, bool TAIL, int MOMENTS, int HD, int KEYS, bool XCH_IN_Q, typename Lds>
__device__ __forceinline__ void stats_body(const ScoreArgs& a, Lds& sm, int unit, int chunk) {
  static_assert(KEYS == KEYS_NONE || (BF16 && !TAIL && !MOMENTS), "keys ride along with the plain sweeps over bf16 caches");
  constexpr bool kSpare = KEYS == KEYS_COS && HD == 128 && NB >= 7;  // see KEYS above
  constexpr int THREADS = kSweepThreads<BF16, NB, HD>, WAVES = THREADS / 64, STEP = THREADS / 2;  // STEP: tokens between two blocks of a wave
  constexpr bool kCentred = MOMENTS == MOMENTS_CENTRED;
  static_assert(!kCentred || (BF16 && !TAIL), "the causal tail and fp32 caches take the sums relative to the first query");
  constexpr int NG = BF16 || MOMENTS ? kGroup<NB> : NB, QS = Tr<BF16, HD>::kQStride;
  extern __shared__ __align__(16) char qlds[];
  auto xch_at = [&](int w, int n) __attribute__((always_inline)) -> float2& {
    if constexpr (XCH_IN_Q)
      return ((float2*)qlds)[w * NB * 32 + n];
    else
      return sm.xch[w][n];
  };
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T_all = seq_len(a.d, a.seq_lens, b), t_end = causal_t_end(a, T_all, CAUSAL);
  const int T = TAIL ? T_all : t_end;
  const int len = chunk_len(a, T_all);
  const int c0 = TAIL ? t_end : chunk * len;
  if (c0 >= T) return;
  const int t_lim = TAIL ? T : min(T, c0 + len);  // the tail (at most W + 31 keys) may be longer than a chunk
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hf = lane >> 5;
  const int t_vis0 = T_all - a.d.W;  // newest key visible to the oldest query of the window
  uint4 av0[Tr<BF16, HD>::kAVecs], av1[Tr<BF16, HD>::kAVecs];
  const int32_t* blk = nullptr;  // paged caches: this chunk's block numbers, staged once
  if (a.k.layout == AMS_LAYOUT_PAGED) {
    stage_blocks<THREADS>(a, b, c0, t_lim, sm.blk);
    blk = sm.blk;
  }
  if (c0 + wave * 32 < t_lim) load_a<BF16, HD>(a, l, b, h, c0 + wave * 32, T, lane, av0, blk, c0);
  const float q_top = load_q<BF16, NB, HD, THREADS>(a, l, b, h, qlds);
  // (not in sm: within one object the write of a block's lengths orders the reads around it; 2423 -> 2386 us per step for the mean
  // cosines of 256 units of 32768 positions, 256 queries)
  __shared__ uint4 ident[KEYS ? 2 : 1][KEYS ? 64 : 1];
  __shared__ __align__(16) double inv_len[KEYS == KEYS_COS ? 4 : 1][KEYS ? 32 : 1];
  __shared__ double ksum_sm[KEYS ? 8 : 1][KEYS ? HD : 1];
  double ksum[KEYS ? HD / 32 : 1];
  if constexpr (KEYS != KEYS_NONE) {
    if (threadIdx.x < 128) {
      const int p = threadIdx.x >> 6, n = lane & 31, one = n - 16 * hf - 8 * p;  // which of the 8 entries is 1
      uint32_t v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (one == 2 * j ? 0x3F80u : 0u) | (one == 2 * j + 1 ? 0x3F800000u : 0u);
      ident[p][lane] = make_uint4(v[0], v[1], v[2], v[3]);
    }
#pragma unroll
    for (int cb = 0; cb < HD / 32; ++cb) ksum[cb] = 0.0;
  }
  const int key_exp = settle_q<BF16, NB, HD, THREADS>(a, l, b, h, qlds, q_top);
  float m[NB], z[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m[nb] = kNegInit;
    z[nb] = 0.f;
  }
  const float c2 = a.c2;
  float* g_row = MOMENTS ? a.g + (int64_t)unit * a.d.t_stride : nullptr;
  if constexpr (kCentred) {
    constexpr int PAIRS = HD / 2, PARTS = kThreads / PAIRS;
    double2* sums = (double2*)sm.g;
    const int pair = threadIdx.x % PAIRS;
    double2 t = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int n = threadIdx.x / PAIRS; n < a.d.N; n += PARTS) {
      const uint32_t v = *(const uint32_t*)(qlds + n * QS + pair * 4);
      t.x += (double)__uint_as_float(v << 16);
      t.y += (double)__uint_as_float(v & 0xFFFF0000u);
    }
    sums[threadIdx.x] = t;
    __syncthreads();
    if (threadIdx.x < PAIRS) {
      for (int p = 1; p < PARTS; ++p) {
        t.x += sums[p * PAIRS + pair].x;
        t.y += sums[p * PAIRS + pair].y;
      }
      const float x[2] = {(float)(-t.x / (double)a.d.N), (float)(-t.y / (double)a.d.N)};
      uint32_t term[3] = {0, 0, 0};
      bool cut = false;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        float r = x[e];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const uint32_t h = __float_as_uint(r) & 0xFFFF0000u;
          term[j] |= e ? h : h >> 16;
          r -= __uint_as_float(h);
        }
        cut |= r != 0.f;
      }
      const int any_cut = __any(cut);
      if (threadIdx.x == 0) sm.mean_cut = any_cut;
#pragma unroll
      for (int j = 0; j < 3; ++j) *(uint32_t*)(sm.mean + j * HD * 2 + pair * 4) = term[j];
    }
    __syncthreads();
  }
  auto block_of = [&](const uint4 (&av)[Tr<BF16, HD>::kAVecs], int t0, auto ragged_c, auto centred_c) __attribute__((always_inline)) {
    constexpr bool ragged = decltype(ragged_c)::value;  // the block reaches past the end of the cache
    constexpr bool centred = kCentred && decltype(centred_c)::value;
    // the query fragments are re-read from LDS for every block: keeping them in registers across
    // blocks would cost more registers than the reads cost time, so their address is made opaque
    int qoff = 0;
    asm volatile("" : "+s"(qoff));
    float ref[16], s1[16], s2[16];
    floatx16 centre;  // minus the mean logit of every token
    if constexpr (centred) {
#pragma unroll
      for (int i = 0; i < 16; ++i) centre[i] = s2[i] = 0.f;
      const char* mb = sm.mean + qoff + hf * HD;
#pragma unroll
      for (int j = 2; j >= 0; --j)  // smallest terms first
#pragma unroll
        for (int ks = 0; ks < Tr<BF16, HD>::kAVecs; ++ks)
          centre = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[ks]),
                                                           __builtin_bit_cast(bf16x8, *(const uint4*)(mb + j * HD * 2 + ks * 16)),
                                                           centre, 0, 0, 0);
    }
    // the vector work on one column block of logits
    auto col_moments = [&](floatx16& acc, int nb) __attribute__((always_inline)) {
      if constexpr (centred) {
        // padded query columns do not count; the first ones are real with every N that takes NB column blocks
        const bool real = nb < kFullBlocks<NB> || nb * 32 + (lane & 31) < a.d.N;
#pragma unroll
        for (int i = 0; i < 16; ++i) s2[i] = __builtin_fmaf(real ? acc[i] : 0.f, acc[i], s2[i]);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] -= centre[i];  // the logit itself
        return;
      }
      if (nb == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          // the half wave's first lane holds the logit against query 0 of the rows this lane owns
          const float r0 = __builtin_amdgcn_readlane(acc[i], 0), r1 = __builtin_amdgcn_readlane(acc[i], 32);
          ref[i] = hf ? r1 : r0;
          s1[i] = s2[i] = 0.f;
        }
      }
      const bool real = nb * 32 + (lane & 31) < a.d.N;  // padded query columns do not count
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float dlt = real ? acc[i] - ref[i] : 0.f;
        s1[i] += dlt;
        s2[i] = __builtin_fmaf(dlt, dlt, s2[i]);
      }
    };
    auto col_stats = [&](floatx16& acc, int nb) __attribute__((always_inline)) {
      if (TAIL) {
        // this column's query sees the keys up to lim (< T, so rows past the end are covered too)
        const int lim = t_vis0 + (nb * 32 + (lane & 31)) % a.d.W;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = (t0 + acc_row(i, hf) > lim) ? -INFINITY : acc[i];
      } else if (ragged) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = (t0 + acc_row(i, hf) >= T) ? -INFINITY : acc[i];
      }
      float mr = acc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mr = fmaxf(mr, acc[i]);
      const float mx = fmaxf(m[nb], mr * c2);  // c2 > 0: the maximum commutes with the scale
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i], c2, -mx));
      z[nb] = __builtin_fmaf(z[nb], __builtin_amdgcn_exp2f(m[nb] - mx), sum);
      m[nb] = mx;
    };
    if constexpr (kPipe<BF16, NB, TAIL> && !kSpare && !ragged) {
      constexpr int NV = Tr<BF16, HD>::kAVecs;
      const char* qb = qlds + qoff + (lane & 31) * QS + (lane >> 5) * (Tr<BF16, HD>::kRowBytes / 2);
      uint4 bq[2][NV];
      floatx16 acc2[2];
      col_frags<BF16, HD>(qb, bq[0]);
      col_frags<BF16, HD>(qb + 32 * QS, bq[1]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (centred) acc2[0] = centre;
      col_mma<BF16, HD, !centred>(av, bq[0], acc2[0]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        __builtin_amdgcn_sched_barrier(0);
        if (nb + 2 < NB) col_frags<BF16, HD>(qb + (nb + 2) * 32 * QS, bq[nb & 1]);
        if (nb + 1 < NB) {
          if constexpr (centred) acc2[(nb + 1) & 1] = centre;
          col_mma<BF16, HD, !centred>(av, bq[(nb + 1) & 1], acc2[(nb + 1) & 1]);
        }
        if (MOMENTS) col_moments(acc2[nb & 1], nb);
        col_stats(acc2[nb & 1], nb);
        if (nb + 2 < NB)
          col_hints<NV, MOMENTS ? 10 : 6, 2, true>();
        else if (nb + 1 < NB)
          col_hints<NV, MOMENTS ? 10 : 6, 2, false>();
      }
    } else if constexpr (kSpare) {
      auto group = [&](auto g0_c) __attribute__((always_inline)) {
        constexpr int g0 = decltype(g0_c)::value, n = NB - g0 < 4 ? NB - g0 : 4;
        floatx16 acc[n];
        tile_mma<BF16, n, HD>(av, qlds + qoff + g0 * 32 * QS, lane, acc);
#pragma unroll
        for (int k = 0; k < n; ++k) col_stats(acc[k], g0 + k);
      };
      group(std::integral_constant<int, 0>{});
      group(std::integral_constant<int, 4>{});
    } else {
      constexpr int n = kCentred && !centred ? 1 : NG;  // the rare second walk takes as few registers as it can
#pragma unroll
      for (int g0 = 0; g0 < NB; g0 += n) {
        floatx16 acc[n];
        if constexpr (centred) {
#pragma unroll
          for (int k = 0; k < n; ++k) acc[k] = centre;
        }
        if (!BF16 && g0 > 0) forget_terms(av);
        tile_mma<BF16, n, HD, !centred, !MOMENTS && !TAIL>(av, qlds + qoff + g0 * 32 * QS, lane, acc, key_exp);
        if (MOMENTS) {
#pragma unroll
          for (int k = 0; k < n; ++k) col_moments(acc[k], g0 + k);
        }
#pragma unroll
        for (int k = 0; k < n; ++k) col_stats(acc[k], g0 + k);
        if (TAIL) __builtin_amdgcn_sched_barrier(0);
      }
    }
    // The sums stay here: sunk past the store of g below they keep the logits of all column blocks (179 registers spilled with 256
    // queries, 128 channels; with 64 channels 727 us per step with this and 759 without, 256 units of 32768, 128 queries; with up to
    // four blocks of 128 channels 1 % more with it).
    if constexpr (CAUSAL && MOMENTS && (kPipe<BF16, NB, TAIL> || HD == 64)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(z[nb]));
    }
    if constexpr (KEYS != KEYS_NONE)
      add_keys<HD, KEYS == KEYS_COS>(av, ident, inv_len[KEYS == KEYS_COS ? wave : 0], lane, ragged ? T - t0 : 32, ksum);
    if constexpr (centred) {
      const int c = lane & 31, t = t0 + acc_row(c >> 1, hf);
      // the variance's share of every lane, and the mean (the same in all of them) from the first one
      const float k_var = 0.5f * a.inv_sqrt_d * a.inv_sqrt_d / (float)a.d.N, k_mean = c == 0 ? -a.inv_sqrt_d / k_var : 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s2[i] = __builtin_fmaf(centre[i], k_mean, s2[i]);
      const float e = reduce16_over32(s2, c) * k_var;
      if ((c & 1) == 0 && t < T_all) sm.g[t - c0] = e;
    } else if (MOMENTS) {
      const int c = lane & 31;
      float rr[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) rr[i] = c == 0 ? ref[i] : 0.f;
      const float inv_n = 1.f / (float)a.d.N;
      const float r_tok = reduce16_over32(rr, c);            // the reference of token c >> 1
      const float d_mean = reduce16_over32(s1, c) * inv_n;   // mean of s - r
      const float d_sq = reduce16_over32(s2, c) * inv_n;     // mean of (s - r)^2
      const int t = t0 + acc_row(c >> 1, hf);
      if ((c & 1) == 0 && t < T_all)
        sm.g[t - c0] = (r_tok + d_mean) * a.inv_sqrt_d + 0.5f * (d_sq - d_mean * d_mean) * (a.inv_sqrt_d * a.inv_sqrt_d);
    }
  };
  auto block = [&](const uint4 (&av)[Tr<BF16, HD>::kAVecs], int t0) __attribute__((always_inline)) {
    // (the plain blocks in front of a tail end at a multiple of 32: without the ragged form next to them the kernels that carry a
    // tail take no more registers than those without.  us per step with it and without: 476 and 462 for 64 fp32 units of 16384, 128
    // queries; 2155 and 1904 for 256 units of 32768, expected attention, 256 queries, where 23 registers spilled)
    if (!(CAUSAL && !TAIL) && t0 + 32 > T)
      block_of(av, t0, std::true_type{}, std::true_type{});
    else
      block_of(av, t0, std::false_type{}, std::true_type{});
  };
  // this wave's blocks: every WAVES-th block of 32 tokens up to the end of the chunk (or of the cache)
#pragma unroll 1
  for (int t0 = c0 + wave * 32; t0 < t_lim; t0 += (TAIL ? 1 : 2) * STEP) {
    if constexpr (TAIL) {  // a wave has one block, seldom more: no second buffer
      block(av0, t0);
      if (t0 + STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + STEP, T, lane, av0, blk, c0);
      continue;
    }
    if (t0 + STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + STEP, T, lane, av1, blk, c0);
    block(av0, t0);
    if (t0 + STEP >= t_lim) break;
    if (t0 + 2 * STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + 2 * STEP, T, lane, av0, blk, c0);
    block(av1, t0 + STEP);
  }
  if constexpr (kCentred) {
    // A key with an infinite entry has no finite centre, and its logits, minus infinity where the queries of that channel have
    // one sign, are lost; and below 2^-109 the smallest numbers that bf16 has cut the terms of the mean query short (queries of
    // 2^-118: 4e-5 of the score's terms).  Then this wave's blocks again, with the sums relative to the first query.
    float t = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) t = __builtin_fmaf(z[nb], 0.f, t);
    if (__builtin_expect(__any(t != 0.f) || sm.mean_cut, 0)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        m[nb] = kNegInit;
        z[nb] = 0.f;
      }
#pragma unroll 1
      for (int t0 = c0 + wave * 32; t0 < t_lim; t0 += STEP) {
        load_a<BF16, HD>(a, l, b, h, t0, T, lane, av0, blk, c0);
        block_of(av0, t0, std::true_type{}, std::false_type{});
      }
    }
  }
  if (XCH_IN_Q) __syncthreads();  // the query window is used up
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float m2 = __shfl_xor(m[nb], 32), z2 = __shfl_xor(z[nb], 32);
    const float M = fmaxf(m[nb], m2);
    // lower half first so that both halves compute the same value
    const float zl = hf ? z2 : z[nb], ml = hf ? m2 : m[nb], zh = hf ? z[nb] : z2, mh = hf ? m[nb] : m2;
    const float Z = zl * __builtin_amdgcn_exp2f(ml - M) + zh * __builtin_amdgcn_exp2f(mh - M);
    if (hf == 0) xch_at(wave, nb * 32 + (lane & 31)) = make_float2(M, Z);
  }
  if constexpr (KEYS != KEYS_NONE) {
    // half waves side by side, added up in a fixed order
#pragma unroll
    for (int cb = 0; cb < HD / 32; ++cb) ksum_sm[wave * 2 + hf][key_channel<HD>(cb, lane & 31)] = ksum[cb];
    __syncthreads();
    if (threadIdx.x < HD) {
      double t = 0.0;
#pragma unroll
      for (int r = 0; r < 8; ++r) t += ksum_sm[r][threadIdx.x];
      a.ksum[((int64_t)unit * a.n_chunks + chunk) * HD + threadIdx.x] = t;
    }
  }
  __syncthreads();
  if (MOMENTS)
    for (int t = c0 + threadIdx.x; t < t_lim; t += THREADS) g_row[t] = sm.g[t - c0];
  if (MOMENTS && !TAIL && a.soft) softmax_part<THREADS>(sm.g, t_lim - c0, a.soft + (int64_t)unit * a.n_chunks + chunk);
  for (int n = threadIdx.x; n < NB * 32; n += THREADS) {
    float M = kNegInit;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, xch_at(w, n).x);
    float Z = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) Z += xch_at(w, n).y * __builtin_amdgcn_exp2f(xch_at(w, n).x - M);
    // the tail's entry follows those of the chunks
    const int slot = TAIL ? (t_end + len - 1) / len : chunk;
    a.part[((int64_t)unit * (a.n_chunks + 1) + slot) * a.n_pad + n] = make_float2(M, Z);
  }
}

// CAUSAL: the last rows of the grid take the tails of the units (moment sums relative to the first query).
template <bool BF16, int NB, bool CAUSAL, int MOMENTS, int HD, int KEYS = KEYS_NONE>
__global__ __launch_bounds__((kSweepThreads<BF16, NB, HD>), (BF16 && NB <= 4 && !MOMENTS && KEYS != KEYS_COS) ? AMS_SCORE_MIN_WAVES : 2) void score_stats_kernel(ScoreArgs a) {
  constexpr bool kXchInQ = MOMENTS == MOMENTS_CENTRED;
  __shared__ StatsLds<BF16, NB, MOMENTS, HD, KEYS> sm;
  int unit, chunk;
  const bool tail = sweep_tile<CAUSAL>(a, false, unit, chunk);
  if constexpr (CAUSAL) {
    if (tail) {
      if (chunk < 0) return;
      stats_body<BF16, NB, CAUSAL, true, MOMENTS ? MOMENTS_FIRST : MOMENTS_NONE, HD, KEYS_NONE, kXchInQ>(a, sm, unit, chunk);
      return;
    }
  }
  stats_body<BF16, NB, CAUSAL, false, MOMENTS, HD, KEYS, kXchInQ>(a, sm, unit, chunk);
}

// What the second sweep needs of query n: reference, weight of its shares in u and in the last-query g, whether it exists.
// last: the last-query score is wanted.
__device__ __forceinline__ float4 query_weights(const ScoreArgs& a, int n, int T, float M, double Z, bool causal, bool last) {
  const bool real = n < a.d.N;
  // causal window on a cache shorter than the window: a query before position 0 does not exist
  const bool exists = real && (!causal || T - a.d.W + (n % a.d.W) >= 0);
  const bool newest = last && exists && (n % a.d.W) == a.d.W - 1;
  return make_float4(M, exists ? (float)(1.0 / ((double)a.d.N * Z)) : 0.f, newest ? (float)(1.0 / ((double)a.d.G * Z)) : 0.f,
                     real ? 1.f : 0.f);
}

// ---------------------------------------------------------------------------------------------
// Sweep 2: u[t] = sum_n exp2(x[n][t] - M_n) / (N Z_n), and g for the softmax-based scorers.
// ---------------------------------------------------------------------------------------------
// Merges a unit's chunk statistics inside the second sweep (launches of few workgroups, where a reduction kernel of its own
// costs more than every workgroup reading them again): weights of query n -> ((float4*)sm)[n], sm of 4 KB; and the sums of
// the chunk's credit before the update, per wave -> c_sm.
template <int THREADS, bool CAUSAL, bool LAST>
__device__ __forceinline__ void fold_stats(const ScoreArgs& a, int unit, int c0, int t_lim, int T, char* sm, double* c_sm) {
  double* pz = (double*)sm;
  float* pm = (float*)(sm + THREADS * sizeof(double));
  double cs = 0.0;
  if (a.vc_part && a.credit) {
    const float* c_row = a.credit + (int64_t)unit * a.d.t_stride;
#pragma unroll 4
    for (int t = c0 + threadIdx.x; t < t_lim; t += THREADS) cs += (double)c_row[t];
  }
  const int len = chunk_len(a, T), nch = (causal_t_end(a, T, CAUSAL) + len - 1) / len + (CAUSAL ? 1 : 0);
  const int parts = THREADS / a.n_pad, n = threadIdx.x % a.n_pad, part = threadIdx.x / a.n_pad;
  if (part < parts) {
    const float2* p = a.part + (int64_t)unit * (a.n_chunks + 1) * a.n_pad + n;
    float M = kNegInit;
    double Z = 0.0;
    for (int first = part; first < nch; first += 8 * parts) {  // eight entries in flight
      float2 s[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        s[i] = first + i * parts < nch ? p[(int64_t)(first + i * parts) * a.n_pad] : make_float2(kNegInit, 0.f);
      float mx = M;
#pragma unroll
      for (int i = 0; i < 8; ++i) mx = fmaxf(mx, s[i].x);
      Z *= (double)__builtin_amdgcn_exp2f(M - mx);
#pragma unroll
      for (int i = 0; i < 8; ++i) Z += (double)s[i].y * (double)__builtin_amdgcn_exp2f(s[i].x - mx);
      M = mx;
    }
    pm[threadIdx.x] = M;
    pz[threadIdx.x] = Z;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) cs += __shfl_xor(cs, o);
  if ((threadIdx.x & 63) == 0) c_sm[threadIdx.x >> 6] = cs;
  __syncthreads();
  float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
  if ((int)threadIdx.x < a.n_pad) {
    float M = kNegInit;
    for (int q = 0; q < parts; ++q) M = fmaxf(M, pm[q * a.n_pad + n]);
    double Z = 0.0;
    for (int q = 0; q < parts; ++q) Z += pz[q * a.n_pad + n] * (double)__builtin_amdgcn_exp2f(pm[q * a.n_pad + n] - M);
    f = query_weights(a, n, T, M, Z, CAUSAL, LAST);
  }
  __syncthreads();
  if ((int)threadIdx.x < a.n_pad) ((float4*)sm)[threadIdx.x] = f;
  __syncthreads();
}

// TAIL (causal window, blocks from t_end on): a (query, key) pair the mask hides adds nothing, and
// every observation a key is missing counts as the largest share it got.
template <bool BF16, int NB, int MODE, int HD, int KEYS, bool FOLD>
struct UsageLds {
  static constexpr int kWaves = kSweepThreads<BF16, NB, HD> / 64;
  // u (and the last-query g) of the chunk are collected in LDS and written once at the end: stores
  // scattered through the sweep cost the key stream 7 % of its rate
  // (last query with 8 column blocks: LDS is needed for the query window)
  static constexpr bool kBufG = KEYS != KEYS_NONE || ((MODE == MODE_LAST || MODE == MODE_LAST_LANES) && NB <= 7);
  static constexpr int kBuf = KEYS != KEYS_NONE || !BF16 ? kKeysChunk : kScoreChunk;
  __align__(16) float u[kBuf];  // (fold_stats uses its head as doubles and float4)
  float g[kBufG ? kBuf : 1];
  double c[FOLD ? kWaves : 1], v[kWaves], k2[2];
  int32_t blk[kScoreChunk / 16];  // paged caches: this chunk's block numbers
};

template <bool BF16, int NB, int MODE, bool CAUSAL, bool TAIL, int HD, int KEYS, bool FOLD, typename Lds>
__device__ __forceinline__ void usage_body(const ScoreArgs& a, Lds& sm, int unit, int chunk) {
  constexpr int THREADS = kSweepThreads<BF16, NB, HD>, WAVES = THREADS / 64, STEP = THREADS / 2;  // STEP: tokens between two blocks of a wave
  constexpr int NG = TAIL ? 1 : BF16 ? kGroup<NB> : NB;  // (the mask and the maxima of the tail take registers)
  constexpr int QS = Tr<BF16, HD>::kQStride;
  extern __shared__ __align__(16) char qlds[];
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T_all = seq_len(a.d, a.seq_lens, b), t_end = causal_t_end(a, T_all, CAUSAL);
  const int T = TAIL ? T_all : t_end;
  const int len = chunk_len(a, T_all);
  const int c0 = TAIL ? t_end : chunk * len;
  if (c0 >= T) return;
  const int t_lim = TAIL ? T : min(T, c0 + len);  // the tail (at most W + 31 keys) may be longer than a chunk
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hf = lane >> 5, c = lane & 31;
  const int t_vis0 = T_all - a.d.W;  // newest key visible to the oldest query of the window
  uint4 av0[Tr<BF16, HD>::kAVecs], av1[Tr<BF16, HD>::kAVecs];
  const int32_t* blk = nullptr;  // paged caches: this chunk's block numbers, staged once
  if (a.k.layout == AMS_LAYOUT_PAGED) {
    stage_blocks<THREADS>(a, b, c0, t_lim, sm.blk);
    blk = sm.blk;
  }
  if (c0 + wave * 32 < t_lim) load_a<BF16, HD>(a, l, b, h, c0 + wave * 32, T, lane, av0, blk, c0);
  const float q_top = load_q<BF16, NB, HD, THREADS>(a, l, b, h, qlds);
  // KEYS: the mean key (or the sum of the unit vectors) as three bf16 terms that add up to its fp32 value, and a row of
  // zeros, behind the query window
  char* krow = qlds + NB * 32 * QS;
  if constexpr (KEYS != KEYS_NONE) {
    if (threadIdx.x < 128) {
      double k = 0.0;
      if (threadIdx.x < HD) {
        const double* ks = a.ksum + (int64_t)unit * a.n_chunks * HD + threadIdx.x;
        if (FOLD) {
          const int nch = (T + len - 1) / len;
#pragma unroll 8
          for (int i = 0; i < nch; ++i) k += ks[(int64_t)i * HD];
        } else {
          k = *ks;
        }
        if (KEYS == KEYS_MEAN) k /= (double)T;
        const float x = (float)k;
        const uint32_t hi = __float_as_uint(x) & 0xFFFF0000u;
        const float r1 = x - __uint_as_float(hi);
        const uint32_t mid = __float_as_uint(r1) & 0xFFFF0000u;
        const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid));
        uint16_t* row = (uint16_t*)krow + threadIdx.x;
        row[0] = (uint16_t)(hi >> 16);
        row[QS / 2] = (uint16_t)(mid >> 16);
        row[QS] = (uint16_t)(lo >> 16);
        row[QS / 2 * 3] = 0;
      }
      double k2 = k * k;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) k2 += __shfl_xor(k2, o);
      // an infinite key: the identity product spreads NaN to the channels next to it, where the sum is none
      if (__ballot(isinf(k))) k2 = INFINITY;
      if (lane == 0) sm.k2[wave] = k2;
    }
  }
  const int key_exp = settle_q<BF16, NB, HD, THREADS>(a, l, b, h, qlds, q_top);
  const double kbar2 = KEYS != KEYS_MEAN                            ? 0.0
                       : isinf(sm.k2[0]) || isinf(sm.k2[1]) ? INFINITY
                                                            : sm.k2[0] + sm.k2[1];  // squared length of the mean key
  const double inv_others = KEYS == KEYS_COS && T > 1 ? 1.0 / (double)(T - 1) : 0.0;
  float* u_row = a.u + (int64_t)unit * a.d.t_stride;
  float* g_row = a.g ? a.g + (int64_t)unit * a.d.t_stride : nullptr;
  const float c2 = a.c2;
  constexpr bool kBufG = Lds::kBufG;
  float4 f[NB];
  if constexpr (FOLD) {
    fold_stats<THREADS, CAUSAL, MODE == MODE_LAST>(a, unit, c0, t_lim, T_all, (char*)sm.u, sm.c);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) f[nb] = ((const float4*)sm.u)[nb * 32 + c];
    __syncthreads();
  } else {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) f[nb] = a.fin[(int64_t)unit * a.n_pad + nb * 32 + c];
  }
  [[maybe_unused]] const int log2_w = 31 - __clz(a.d.W);  // MODE_LAST_LANES: of a power of two
  if (MODE == MODE_LAST_LANES) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) f[nb].y *= (float)a.d.W;
  }
  float v_part = 0.f;  // this lane's share of sum(max(u,0)+eps): one term per block of 32 keys of this wave (32 blocks per chunk)
  auto block = [&](const uint4 (&av)[Tr<BF16, HD>::kAVecs], int t0) __attribute__((always_inline)) {
    float pu[16], pg[16], pm[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) pu[i] = pg[i] = pm[i] = 0.f;
    float rg = 0.f;
    constexpr bool masked = TAIL;
    int qoff = 0;  // see the first sweep: the query fragments are re-read per block on purpose
    asm volatile("" : "+s"(qoff));
    auto col_usage = [&](const floatx16& acc, int nb) __attribute__((always_inline)) {
      if (masked) {
        const int lim = t_vis0 + (nb * 32 + c) % a.d.W;  // newest key this column's query sees
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i], c2, -f[nb].x));
          const bool sees = t0 + acc_row(i, hf) <= lim;
          const float share = sees ? f[nb].y * e : 0.f;
          pu[i] += share;
          pm[i] = fmaxf(pm[i], share);
          if (!BF16 && MODE == MODE_LAST) pg[i] += sees ? f[nb].z * e : 0.f;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i], c2, -f[nb].x));
          pu[i] = __builtin_fmaf(f[nb].y, e, pu[i]);
          if (MODE == MODE_LAST) pg[i] = __builtin_fmaf(f[nb].z, e, pg[i]);
        }
      }
    };
    if constexpr (kPipe<BF16, NB, TAIL>) {
      constexpr int NV = Tr<BF16, HD>::kAVecs;
      const char* qb = qlds + qoff + (lane & 31) * QS + (lane >> 5) * (Tr<BF16, HD>::kRowBytes / 2);
      uint4 bq[2][NV];
      floatx16 acc2[2];
      col_frags<BF16, HD>(qb, bq[0]);
      col_frags<BF16, HD>(qb + 32 * QS, bq[1]);
      __builtin_amdgcn_sched_barrier(0);
      col_mma<BF16, HD>(av, bq[0], acc2[0]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        __builtin_amdgcn_sched_barrier(0);
        if (nb + 2 < NB) col_frags<BF16, HD>(qb + (nb + 2) * 32 * QS, bq[nb & 1]);
        if (nb + 1 < NB) col_mma<BF16, HD>(av, bq[(nb + 1) & 1], acc2[(nb + 1) & 1]);
        col_usage(acc2[nb & 1], nb);
        if (nb + 2 < NB)
          col_hints<NV, MODE == MODE_LAST ? 6 : 4, 2, true>();
        else if (nb + 1 < NB)
          col_hints<NV, MODE == MODE_LAST ? 6 : 4, 2, false>();
      }
    } else {
#pragma unroll
      for (int g0 = 0; g0 < NB; g0 += NG) {
        floatx16 acc[NG];
        tile_mma<BF16, NG, HD>(av, qlds + qoff + g0 * 32 * QS, lane, acc, key_exp);
#pragma unroll
        for (int k = 0; k < NG; ++k) col_usage(acc[k], g0 + k);
        if (TAIL) __builtin_amdgcn_sched_barrier(0);
      }
    }
    const int t = t0 + acc_row(c >> 1, hf);
    float ru = reduce16_over32(pu, c);
    if (masked) {
      const int seen = a.d.G * min(a.d.W, T - t);  // (head, query) pairs that see key t
      ru += (float)(a.d.N - seen) * reduce16_over32<true>(pm, c);
      // The products once more, instead of a third sum next to the usage and its maxima, which the bf16 kernels do not have the
      // registers for (27 spilled at 65 to 128 queries, 8 at 256: 108.1 -> 106.9 us per step for 64 units of 8192, 318.6 -> 315.3
      // for 128 of 16000; fp32 kernels, two waves on a SIMD, hold it: 90.4 and 95.6 with the products twice, 8 units of 8192).
      if constexpr (BF16 && MODE == MODE_LAST) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          floatx16 acc[1];
          tile_mma<BF16, 1, HD>(av, qlds + qoff + nb * 32 * QS, lane, acc, key_exp);
#pragma unroll
          for (int i = 0; i < 16; ++i)  // (the newest queries see every key)
            pg[i] += f[nb].z != 0.f ? f[nb].z * __builtin_amdgcn_exp2f(__builtin_fmaf(acc[0][i], c2, -f[nb].x)) : 0.f;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (MODE == MODE_LAST_LANES) ru = ldexpf(ru, -log2_w);
    if (MODE == MODE_MEAN) rg = ru;
    if constexpr (KEYS != KEYS_NONE) {
      const float n2 = __shfl(key_norm2(key_gram<HD>(av), c), hf * 32 + acc_row(c >> 1, hf));  // of token t
      // column 3 g + j holds term j of the mean key in the channels of step g only: every column adds up 16 products, and
      // the columns are added by halves below, instead of one long chain of additions
      uint4 kq[Tr<BF16, HD>::kAVecs];
      const char* kb = krow + qoff + hf * (Tr<BF16, HD>::kRowBytes / 2);
#pragma unroll
      for (int ks = 0; ks < Tr<BF16, HD>::kAVecs; ++ks)
        kq[ks] = *(const uint4*)(kb + (c / 3 == ks ? c % 3 : 3) * QS + ks * 16);
      floatx16 acc;
      col_mma<BF16, HD>(av, kq, acc);
      float pk[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) pk[i] = acc[i];
      const double dot = (double)reduce16_over32(pk, c);
      if (KEYS == KEYS_MEAN) {  // minus the cosine to the mean key
        const double den2 = (double)n2 * kbar2;
        rg = den2 > 0.0 ? (float)(-dot * rsqrt(den2)) : 0.f;
      } else {  // mean cosine to the other keys
        rg = (n2 > 0.f && T > 1) ? (float)((dot * rsqrt((double)n2) - 1.0) * inv_others) : 0.f;
      }
    }
    if (MODE == MODE_LAST) rg = reduce16_over32(pg, c);
    if (MODE == MODE_LAST_LANES) rg = newest_lanes(pu, c, a.d.W);
    if ((c & 1) == 0 && t < T) {
      sm.u[t - c0] = ru;
      if (kBufG)
        sm.g[t - c0] = rg;
      else if (g_row)
        g_row[t] = rg;
      v_part += fmaxf(ru, 0.f) + a.eps;
    }
  };
  // this wave's blocks: every WAVES-th block of 32 tokens up to the end of the chunk (or of the cache)
#pragma unroll 1
  for (int t0 = c0 + wave * 32; t0 < t_lim; t0 += (TAIL ? 1 : 2) * STEP) {
    if constexpr (TAIL) {  // a wave has one block, seldom more: no second buffer
      block(av0, t0);
      if (t0 + STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + STEP, T, lane, av0, blk, c0);
      continue;
    }
    if (t0 + STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + STEP, T, lane, av1, blk, c0);
    block(av0, t0);
    if (t0 + STEP >= t_lim) break;
    if (t0 + 2 * STEP < t_lim) load_a<BF16, HD>(a, l, b, h, t0 + 2 * STEP, T, lane, av0, blk, c0);
    block(av1, t0 + STEP);
  }
  __syncthreads();
  for (int t = c0 + threadIdx.x; t < t_lim; t += THREADS) {
    u_row[t] = sm.u[t - c0];
    if (kBufG) g_row[t] = sm.g[t - c0];
  }
  if (KEYS == KEYS_COS) softmax_part(sm.g, t_lim - c0, a.soft + (int64_t)unit * a.n_chunks + chunk);
  if (a.vc_part) {  // chunk sums of max(u,0)+eps in a fixed order: lanes, then waves
    double v_acc = (double)v_part;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v_acc += __shfl_xor(v_acc, o);
    if (lane == 0) sm.v[wave] = v_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      // the unit's credit sum (formed between the sweeps) rides in the first chunk's entry
      double c = (!FOLD && chunk == 0 && a.csum) ? a.csum[unit] : 0.0;
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; w += 2) {
        v += sm.v[w] + sm.v[w + 1];
        if (FOLD) c += sm.c[w] + sm.c[w + 1];
      }
      a.vc_part[(int64_t)unit * a.n_chunks + chunk] = make_double2(v, c);
    }
  }
}

template <bool BF16, int NB, int MODE, bool CAUSAL, int HD, int KEYS = KEYS_NONE, bool FOLD = false>
__global__ __launch_bounds__((kSweepThreads<BF16, NB, HD>), (BF16 && NB <= 4) ? AMS_SCORE_MIN_WAVES : 2) void score_usage_kernel(ScoreArgs a) {
  __shared__ UsageLds<BF16, NB, MODE, HD, KEYS, FOLD> sm;
  if (FOLD && a.status && (blockIdx.x | blockIdx.y | threadIdx.x) == 0) *a.status = 0;  // no bounded wait on this path
  // the second sweep walks the cache backwards: what the first sweep read last is still in the
  // memory-side cache (about a tenth of the keys at the headline size)
  int unit, chunk;
  const bool tail = sweep_tile<CAUSAL>(a, true, unit, chunk);
  if constexpr (CAUSAL) {
    if (tail) {
      if (chunk < 0) return;
      usage_body<BF16, NB, MODE, CAUSAL, true, HD, KEYS, FOLD>(a, sm, unit, chunk);
      return;
    }
  }
  usage_body<BF16, NB, MODE, CAUSAL, false, HD, KEYS, FOLD>(a, sm, unit, chunk);
}

// Calls f with the tile of a launch: (bf16 cache, column blocks, channels) as types.
template <typename F>
hipError_t by_tile(int nb, int head_dim, bool bf16, F f) {
  auto by_nb = [&](auto bf16_c, auto hd_c) {
    if (nb <= 1) return f(bf16_c, std::integral_constant<int, 1>{}, hd_c);
    if (nb <= 2) return f(bf16_c, std::integral_constant<int, 2>{}, hd_c);
    if (nb <= 4) return f(bf16_c, std::integral_constant<int, 4>{}, hd_c);
    if constexpr (decltype(bf16_c)::value) {
      if (nb <= 7) return f(bf16_c, std::integral_constant<int, 7>{}, hd_c);
      if (nb <= 8) return f(bf16_c, std::integral_constant<int, 8>{}, hd_c);
    }
    return hipErrorInvalidValue;
  };
  auto by_dtype = [&](auto hd_c) { return bf16 ? by_nb(std::true_type{}, hd_c) : by_nb(std::false_type{}, hd_c); };
  return head_dim == 64 ? by_dtype(std::integral_constant<int, 64>{}) : by_dtype(std::integral_constant<int, 128>{});
}

template <bool BF16, int NB, bool CAUSAL, int HD>
hipError_t launch_stats(const ScoreArgs& a, bool moments, hipStream_t s) {
  const SweepGrid sg = sweep_grid(a.d.units, a.n_chunks, CAUSAL);
  auto launch = [&](auto moments_c) {
    constexpr int M = decltype(moments_c)::value, lds = NB * 32 * Tr<BF16, HD>::kQStride;
    const hipError_t e = ensure_lds<score_stats_kernel<BF16, NB, CAUSAL, M, HD>>(lds);
    if (e != hipSuccess) return e;
    prof_mark("score_stats", s);
    hipLaunchKernelGGL((score_stats_kernel<BF16, NB, CAUSAL, M, HD>), dim3(sg.x, sg.y), dim3(kSweepThreads<BF16, NB, HD>), lds, s, a);
    return hipGetLastError();
  };
  if (!moments) return launch(std::integral_constant<int, MOMENTS_NONE>{});
  if constexpr (BF16 && HD == 64) {
    return launch(std::integral_constant<int, MOMENTS_CENTRED>{});
  } else {
    if constexpr (BF16 && NB == 4)
      if ((int64_t)a.n_chunks * a.d.units >= 512) return launch(std::integral_constant<int, MOMENTS_CENTRED>{});
    return launch(std::integral_constant<int, MOMENTS_FIRST>{});
  }
}

template <bool BF16, int NB, int MODE, bool CAUSAL, int HD>
hipError_t launch_usage(const ScoreArgs& a, hipStream_t s) {
  const SweepGrid sg = sweep_grid(a.d.units, a.n_chunks, CAUSAL);
  auto launch = [&](auto fold_c) {
    constexpr bool F = decltype(fold_c)::value;
    constexpr int lds = NB * 32 * Tr<BF16, HD>::kQStride;
    const hipError_t e = ensure_lds<score_usage_kernel<BF16, NB, MODE, CAUSAL, HD, KEYS_NONE, F>>(lds);
    if (e != hipSuccess) return e;
    prof_mark("score_usage", s);
    hipLaunchKernelGGL((score_usage_kernel<BF16, NB, MODE, CAUSAL, HD, KEYS_NONE, F>), dim3(sg.x, sg.y),
                       dim3(kSweepThreads<BF16, NB, HD>), lds, s, a);
    return hipGetLastError();
  };
  return a.fold ? launch(std::true_type{}) : launch(std::false_type{});
}

// The sweeps over the caches of one kind of window.  The first one and the reduction after it are the same for every scorer; a file
// holds the kernels that it names.
template <bool CAUSAL>
hipError_t first_sweep(const ScoreArgs& a, int nb, int head_dim, bool moments, bool bf16, hipStream_t s) {
  const hipError_t e = by_tile(nb, head_dim, bf16, [&](auto bf16_c, auto nb_c, auto hd_c) {
    return launch_stats<decltype(bf16_c)::value, decltype(nb_c)::value, CAUSAL, decltype(hd_c)::value>(a, moments, s);
  });
  return e != hipSuccess || a.fold ? e : launch_score_reduce(a, s);
}
template <int MODE, bool CAUSAL>
hipError_t second_sweep(const ScoreArgs& a, int nb, int head_dim, bool bf16, hipStream_t s) {
  return by_tile(nb, head_dim, bf16, [&](auto bf16_c, auto nb_c, auto hd_c) {
    return launch_usage<decltype(bf16_c)::value, decltype(nb_c)::value, MODE, CAUSAL, decltype(hd_c)::value>(a, s);
  });
}

// The two plain sweeps with the keys riding along.
template <int NB, int HD, int KEYS, bool FOLD>
hipError_t run_key_sweeps(const ScoreArgs& a, hipStream_t s) {
  constexpr auto usage = score_usage_kernel<true, NB, MODE_MEAN, false, HD, KEYS, FOLD>;
  const int lds = NB * 32 * Tr<true, HD>::kQStride, lds_k = lds + 4 * Tr<true, HD>::kQStride;
  const dim3 grid(a.n_chunks, a.d.units), blk(kThreads);
  hipError_t e;
  if ((e = ensure_lds<score_stats_kernel<true, NB, false, MOMENTS_NONE, HD, KEYS>>(lds)) != hipSuccess) return e;
  if ((e = ensure_lds<usage>(lds_k)) != hipSuccess) return e;
  prof_mark("score_stats", s);
  hipLaunchKernelGGL((score_stats_kernel<true, NB, false, MOMENTS_NONE, HD, KEYS>), grid, blk, lds, s, a);
  if (!FOLD && (e = launch_score_reduce(a, s)) != hipSuccess) return e;
  prof_mark("score_usage", s);
  hipLaunchKernelGGL(usage, grid, blk, lds_k, s, a);
  return hipGetLastError();
}

}  // namespace
}  // namespace ams
#endif
