// Usage u and the softmax-based g of a SHORT cache in one launch (Alg. 1 step 1; Sec. 3.2; Sec. 3.3;
// App. "Compression schedule": after the first event a cache is the kept rows plus the tokens decoded
// since, a few thousand positions).
//
// One workgroup owns a whole unit (at most kScoreChunk positions): it walks the unit's keys once for the
// per-query (max, sum of exp), merges them inside the workgroup, and walks the keys again for the usage --
// the second walk finds the keys in the caches they were just pulled through.  The arithmetic is that of the
// two-sweep kernels (score.hip): the same tiles, the same running statistics, the normaliser in double; what
// goes away are two launches and the trip of the statistics through memory, which is most of the scorer's
// time when an event moves only a couple of megabytes per unit.
#include "mass_cuts.h"
#include "score_tile.h"

namespace ams {
namespace {

constexpr int kUnitThreads = 512, kUnitWaves = kUnitThreads / 64;

// CUTS: the workgroup goes on to the masses, the cuts and the quotas (mass_cuts.h) on the usage that it holds, 4 to 9 us at its end
// for one or two launches of 11 to 17.  us per step without and with: 170.5 and 166.1 (256 units of 2176, 128 queries), 86.9 and
// 82.2 (192 of 4093, 64 channels), 110.3 and 101.8 (832 of 1425, 64 channels), 58.6 and 55.5 (300 of 1024, 8 queries), 407 and 398
// (1224 of 3000, 32 queries).  Only in launches of few rounds (launch_score).
template <bool BF16, int NB, int MODE, int HD, bool CUTS>
__global__ __launch_bounds__(kUnitThreads, (unit_tile_small(BF16, NB, HD) ? 4 : 2)) void score_unit_kernel(ScoreArgs a, MsArgs ms, CutsOut out) {
  constexpr int NG = (BF16 && NB % 2 == 0 && NB >= 4) ? NB / 2 : NB, QS = Tr<BF16, HD>::kQStride, NQ = NB * 32;
  constexpr bool kLast = MODE == MODE_LAST || MODE == MODE_LAST_LANES;
  extern __shared__ __align__(16) char qlds[];
  __shared__ float2 xch[kUnitWaves][NQ];
  __shared__ float4 fin_s[NQ];
  __shared__ __align__(16) float u_sm[kScoreChunk];
  constexpr int kRounds = kScoreChunk / (kUnitThreads * 4);  // runs of four positions per thread
  [[maybe_unused]] __shared__ CutsLds<kUnitThreads, CUTS ? CUTS_UNIT : CUTS_STEP, CUTS ? kRounds : 1> cuts_sm;
  __shared__ float g_sm[kLast ? kScoreChunk : 1];
  __shared__ double2 vc_sm[kUnitWaves];
  const int unit = blockIdx.x;
  if (unit == 0 && threadIdx.x == 0 && a.status) *a.status = 0;  // no bounded wait on this path
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  float cr[kRounds][4];  // the old credit of the unit (for the EMA normaliser)
  auto go_on = [&](double Z, double c_old) __attribute__((always_inline)) {
    if constexpr (CUTS) cuts_body<kUnitThreads, CUTS_UNIT, kRounds>(ms, out.m_used, out, unit, cuts_sm, u_sm, cr, Z, c_old);
  };
  if (T <= 0) {
    go_on(0.0, 0.0);
    return;
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hf = lane >> 5, c = lane & 31;
  uint4 av0[Tr<BF16, HD>::kAVecs], av1[Tr<BF16, HD>::kAVecs];
  constexpr int kStep = kUnitWaves * 32;  // tokens between two blocks of one wave
  if (wave * 32 < T) load_a<BF16, HD>(a, l, b, h, wave * 32, T, lane, av0);
  const float q_top = load_q<BF16, NB, HD, kUnitThreads>(a, l, b, h, qlds);
  // In flight during the walks, 16 bytes at a time also where only the sum is wanted (CUTS = false): us per step with 4-byte loads
  // and with these 306.0 and 301.5 (2048 units of 1024, 64 channels), 799 and 791 (3000 of 1000), 588 and 585 (700 of 4000).
  const bool credit = a.vc_part && a.credit, vec = CUTS ? ms.vec : (a.d.t_stride & 3) == 0 && ((uintptr_t)a.credit & 15) == 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    load_run(a.credit + (int64_t)unit * a.d.t_stride, (r * kUnitThreads + (int)threadIdx.x) * 4, credit ? T : 0, vec, cr[r], 0.f);
  const int key_exp = settle_q<BF16, NB, HD, kUnitThreads>(a, l, b, h, qlds, q_top);
  const float c2 = a.c2;

  // ---- first walk: per query (max, sum exp2) of the scaled logits over this wave's blocks ----
  float m[NB], z[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m[nb] = kNegInit;
    z[nb] = 0.f;
  }
  auto stats_block = [&](const uint4 (&av)[Tr<BF16, HD>::kAVecs], int t0) __attribute__((always_inline)) {
    const bool ragged = t0 + 32 > T;
    int qoff = 0;  // the query fragments are re-read from LDS per block on purpose (registers)
    asm volatile("" : "+s"(qoff));
#pragma unroll
    for (int g0 = 0; g0 < NB; g0 += NG) {
      floatx16 acc[NG];
      tile_mma<BF16, NG, HD>(av, qlds + qoff + g0 * 32 * QS, lane, acc, key_exp);
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const int nb = g0 + k;
        if (ragged) {
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[k][i] = (t0 + acc_row(i, hf) >= T) ? -INFINITY : acc[k][i];
        }
        float mr = acc[k][0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mr = fmaxf(mr, acc[k][i]);
        const float mx = fmaxf(m[nb], mr * c2);  // c2 > 0: the maximum commutes with the scale
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[k][i], c2, -mx));
        z[nb] = __builtin_fmaf(z[nb], __builtin_amdgcn_exp2f(m[nb] - mx), sum);
        m[nb] = mx;
      }
    }
  };
#pragma unroll 1
  for (int t0 = wave * 32; t0 < T; t0 += 2 * kStep) {
    if (t0 + kStep < T) load_a<BF16, HD>(a, l, b, h, t0 + kStep, T, lane, av1);
    stats_block(av0, t0);
    if (t0 + kStep >= T) break;
    if (t0 + 2 * kStep < T) load_a<BF16, HD>(a, l, b, h, t0 + 2 * kStep, T, lane, av0);
    stats_block(av1, t0 + kStep);
  }
  // the second walk's first block travels during the merge
  if (wave * 32 < T) load_a<BF16, HD>(a, l, b, h, wave * 32, T, lane, av0);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float m2 = __shfl_xor(m[nb], 32), z2 = __shfl_xor(z[nb], 32);
    const float M = fmaxf(m[nb], m2);
    // lower half first so that both halves compute the same value
    const float zl = hf ? z2 : z[nb], ml = hf ? m2 : m[nb], zh = hf ? z[nb] : z2, mh = hf ? m[nb] : m2;
    const float Z = zl * __builtin_amdgcn_exp2f(ml - M) + zh * __builtin_amdgcn_exp2f(mh - M);
    if (hf == 0) xch[wave][nb * 32 + c] = make_float2(M, Z);
  }
  __syncthreads();
  if (threadIdx.x < NQ) {  // waves merged in index order, the normaliser in double
    const int n = threadIdx.x;
    float M = kNegInit;
#pragma unroll
    for (int w = 0; w < kUnitWaves; ++w) M = fmaxf(M, xch[w][n].x);
    double Z = 0.0;
#pragma unroll
    for (int w = 0; w < kUnitWaves; ++w) Z += (double)xch[w][n].y * (double)__builtin_amdgcn_exp2f(xch[w][n].x - M);
    const bool real = n < a.d.N;
    const bool newest = real && (n % a.d.W) == a.d.W - 1;
    fin_s[n] = make_float4(M, real ? (float)(1.0 / ((double)(MODE == MODE_LAST_LANES ? a.d.G : a.d.N) * Z)) : 0.f,
                           newest ? (float)(1.0 / ((double)a.d.G * Z)) : 0.f, real ? 1.f : 0.f);
  }
  __syncthreads();

  // ---- second walk: u[t] = sum_n exp2(x[n][t] - M_n) / (N Z_n), and the last-query g ----
  float4 f[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) f[nb] = fin_s[nb * 32 + c];
  [[maybe_unused]] const int log2_w = 31 - __clz(a.d.W);  // MODE_LAST_LANES: of a power of two
  float v_part = 0.f;  // this lane's share of sum(max(u,0)+eps)
  auto usage_block = [&](const uint4 (&av)[Tr<BF16, HD>::kAVecs], int t0) __attribute__((always_inline)) {
    float pu[16], pg[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) pu[i] = pg[i] = 0.f;
    int qoff = 0;
    asm volatile("" : "+s"(qoff));
#pragma unroll
    for (int g0 = 0; g0 < NB; g0 += NG) {
      floatx16 acc[NG];
      tile_mma<BF16, NG, HD>(av, qlds + qoff + g0 * 32 * QS, lane, acc, key_exp);
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const int nb = g0 + k;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[k][i], c2, -f[nb].x));
          pu[i] = __builtin_fmaf(f[nb].y, e, pu[i]);
          if (MODE == MODE_LAST) pg[i] = __builtin_fmaf(f[nb].z, e, pg[i]);
        }
      }
    }
    const int t = t0 + acc_row(c >> 1, hf);
    float ru = reduce16_over32(pu, c);
    if (MODE == MODE_LAST_LANES) ru = ldexpf(ru, -log2_w);
    float rg = ru;
    if (MODE == MODE_LAST) rg = reduce16_over32(pg, c);
    if (MODE == MODE_LAST_LANES) rg = newest_lanes(pu, c, a.d.W);
    if ((c & 1) == 0 && t < T) {
      u_sm[t] = ru;
      if (kLast) g_sm[t] = rg;
      v_part += fmaxf(ru, 0.f) + a.eps;
    }
  };
#pragma unroll 1
  for (int t0 = wave * 32; t0 < T; t0 += 2 * kStep) {
    if (t0 + kStep < T) load_a<BF16, HD>(a, l, b, h, t0 + kStep, T, lane, av1);
    usage_block(av0, t0);
    if (t0 + kStep >= T) break;
    if (t0 + 2 * kStep < T) load_a<BF16, HD>(a, l, b, h, t0 + 2 * kStep, T, lane, av0);
    usage_block(av1, t0 + kStep);
  }
  __syncthreads();
  float* u_row = a.u + (int64_t)unit * a.d.t_stride;
  float* g_row = a.g ? a.g + (int64_t)unit * a.d.t_stride : nullptr;
  for (int t = threadIdx.x; t < T; t += kUnitThreads) {
    u_row[t] = u_sm[t];
    if (g_row) g_row[t] = kLast ? g_sm[t] : u_sm[t];
  }
  if (a.vc_part) {  // the unit's sums of max(u,0)+eps and of the old credit: lanes, then waves, fixed order
    double v_acc = (double)v_part, c_acc = 0.0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) c_acc += (double)cr[r][i];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      v_acc += __shfl_xor(v_acc, o);
      c_acc += __shfl_xor(c_acc, o);
    }
    if (lane == 0) vc_sm[wave] = make_double2(v_acc, c_acc);
    __syncthreads();
    if (CUTS || threadIdx.x == 0) {
      double2 t = vc_sm[0];
      for (int w = 1; w < kUnitWaves; ++w) {
        t.x += vc_sm[w].x;
        t.y += vc_sm[w].y;
      }
      if constexpr (CUTS)
        go_on(t.x, t.y);
      else
        a.vc_part[unit] = t;
    }
  }
}

template <bool BF16, int NB, int MODE, int HD>
hipError_t launch_unit(const ScoreArgs& a, const UnitCuts* cuts, hipStream_t s) {
  const int lds = NB * 32 * Tr<BF16, HD>::kQStride;
  auto launch = [&](auto cuts_c, const UnitCuts& u) {
    constexpr bool C = decltype(cuts_c)::value;
    const hipError_t e = ensure_lds<score_unit_kernel<BF16, NB, MODE, HD, C>>(lds);
    if (e != hipSuccess) return e;
    prof_mark("score_unit", s);
    hipLaunchKernelGGL((score_unit_kernel<BF16, NB, MODE, HD, C>), dim3(a.d.units), dim3(kUnitThreads), lds, s, a, u.a, u.o);
    return hipGetLastError();
  };
  if (!cuts) return launch(std::false_type{}, UnitCuts{});
  UnitCuts u = *cuts;
  u.o.status = nullptr;  // no bounded wait on this path, and unit 0 clears the word while others would read it
  return launch(std::true_type{}, u);
}

template <bool BF16, int HD>
hipError_t unit_by_nb(const ScoreArgs& a, int nb, int mode, const UnitCuts* cuts, hipStream_t s, bool* ran) {
  *ran = true;
#define AMS_UNIT_CASE(NBV)                                                           \
  if (nb <= NBV) {                                                                   \
    if (mode == MODE_LAST) return launch_unit<BF16, NBV, MODE_LAST, HD>(a, cuts, s);       \
    if (mode == MODE_LAST_LANES) return launch_unit<BF16, NBV, MODE_LAST_LANES, HD>(a, cuts, s); \
    return launch_unit<BF16, NBV, MODE_MEAN, HD>(a, cuts, s);                              \
  }
  AMS_UNIT_CASE(1)
  AMS_UNIT_CASE(2)
  AMS_UNIT_CASE(4)
#undef AMS_UNIT_CASE
  *ran = false;
  return hipSuccess;
}

}  // namespace

// Runs the one-launch scorer when it applies: caches of at most kScoreChunk positions, bf16 or fp32, up to
// 128 queries per KV head, no causal window, mean-window / last-query statistics (the key-diversity scorer
// takes its usage from here too).  *ran = false: the caller uses the two sweeps.
hipError_t launch_score_unit(const ScoreArgs& a, bool bf16, int head_dim, int mode, const UnitCuts* cuts, hipStream_t s, bool* ran) {
  *ran = false;
  if (a.d.t_max > kScoreChunk || a.causal || mode == MODE_EXPECTED || a.n_pad > 128) return hipSuccess;
  const int nb = a.n_pad / 32;
  if (head_dim == 64)
    return bf16 ? unit_by_nb<true, 64>(a, nb, mode, cuts, s, ran) : unit_by_nb<false, 64>(a, nb, mode, cuts, s, ran);
  return bf16 ? unit_by_nb<true, 128>(a, nb, mode, cuts, s, ran) : unit_by_nb<false, 128>(a, nb, mode, cuts, s, ran);
}

}  // namespace ams
