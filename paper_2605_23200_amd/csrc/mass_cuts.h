// What follows the scores of a unit (Sec. 3.2, 3.3; Alg. 1 steps 1-4): masses and credit position by position, the prefix over
// them, cuts, segment masses and quotas.  Used by the kernels of mass_segment.hip (see there) and by the one-launch scorer.
#ifndef AMS_MASS_CUTS_H
#define AMS_MASS_CUTS_H

#include <type_traits>

#include "ams_internal.h"
#include "quota.h"

namespace ams {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kMaxSegments = 1024;

// Sum over the workgroup, same value in every thread, fixed order.
template <int WAVES = kWaves>
__device__ __forceinline__ double block_sum(double v, double* sm) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();  // sm may still be read from a previous call
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) t += sm[w];
  return t;
}

// N consecutive fp32 of a row: 16-byte accesses when the row allows it.
template <int N>
__device__ __forceinline__ void load_run(const float* row, int j0, int T, bool vec, float (&x)[N], float fill) {
  if (vec && j0 + N <= T) {
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
      const float4 v = *reinterpret_cast<const float4*>(row + j0 + 4 * q);
      x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = (j0 + i < T) ? row[j0 + i] : fill;
  }
}
template <int N>
__device__ __forceinline__ void store_run(float* row, int j0, int T, bool vec, const float (&x)[N]) {
  if (vec && j0 + N <= T) {
#pragma unroll
    for (int q = 0; q < N / 4; ++q)
      *reinterpret_cast<float4*>(row + j0 + 4 * q) = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (j0 + i < T) row[j0 + i] = x[i];
  }
}

// Mean of u over the positions t - r .. t + r that exist, for the four positions from t0 on, from one walk over the scores that
// they see; tile[e] is position t0 - r, positions that do not exist hold zeros.
__device__ __forceinline__ void pool_run(const float* tile, int e, int t0, int T, int r, float (&pooled)[4]) {
  const double inv_full = 1.0 / (double)(2 * r + 1);
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  for (int q = 0; q < 2 * r + 4; q += 4) {
    const float4 x4 = *reinterpret_cast<const float4*>(&tile[e + q]);
    const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (q + j >= i && q + j <= i + 2 * r) sum[i] += (double)x[j];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = t0 + i;
    const int n = min(T - 1, t + r) - max(0, t - r) + 1;
    pooled[i] = (float)(n == 2 * r + 1 ? sum[i] * inv_full : sum[i] / (double)n);
  }
}

constexpr int kMaxPoolR = 31;

struct MsArgs {
  Dims d;
  const int32_t* seq_lens;
  int S;             // entries of the per-unit segment arrays
  int K;             // initial segments: thresholds k = 1..K-1 (K == S unless delta > 0)
  double delta;      // > 0: thresholds k*delta; 0: thresholds k/S
  int l_min, l_max;  // delta > 0 only: length rules of the split / merge pass (0 = off)
  int pool_r;        // radius of the average pooling of u before Eq. (1) (0 = off)
  double2* vc_part;  // [units][vc_stride] (sum of max(u,0)+eps, sum of old credit) per vc_tokens positions
  int vc_stride, vc_tokens;
  bool vc_even;      // see VcInfo
  double* sub;       // [units][n_sub] sum of m_used per kSub positions; stage call: pairs (sum, largest prefix inside)
  int n_sub;
  int32_t* bounds;   // [units][S+1]
  bool vec;          // rows of the fp32 vectors are 16-byte aligned
};

// ---- pieces of kSub positions: 16 lanes (one DPP row) with four consecutive positions each ----
constexpr int kSub = 64;
constexpr int kSubLanes = kSub / 4;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {  // lanes without a source read 0
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Inclusive prefix of the piece at this lane's four positions; lane 15's last entry is the piece's total.
__device__ __forceinline__ void sub_scan(const float (&x)[4], double (&p)[4]) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) s += (double)x[i];
  double incl = s;  // row_shr: 1, 2, 4, 8
  incl += dpp_f64<0x111>(incl);
  incl += dpp_f64<0x112>(incl);
  incl += dpp_f64<0x114>(incl);
  incl += dpp_f64<0x118>(incl);
  double run = dpp_f64<0x111>(incl);  // prefix in front of this lane
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    run += (double)x[i];
    p[i] = run;
  }
}

// Normalisers of one unit: its partial sums of max(u,0)+eps and of the old credit, added up by every wave for itself (strided
// over the lanes, then a fixed tree).
struct MassOf {
  double lam, bet, eps, inv_z, inv_csum;
  bool ema;
  __device__ __forceinline__ MassOf(float lambda, float beta, float eps_f, double Z, double c_old)
      : lam((double)lambda), bet((double)beta), eps((double)eps_f), ema(lambda != 0.f) {
    normalise(Z, c_old);
  }
  __device__ __forceinline__ void normalise(double Z, double c_old) {
    inv_z = 1.0 / Z;
    inv_csum = 1.0 / (lam * c_old + (1.0 - lam));
  }
  __device__ __forceinline__ MassOf(const MsArgs& a, int unit, int T, float lambda, float beta, float eps_f)
      : lam((double)lambda), bet((double)beta), eps((double)eps_f), ema(lambda != 0.f) {
    const int tokens = a.vc_even && T != a.d.t_max ? even_chunk(T, a.vc_stride) : a.vc_tokens;
    const int nvc = (T + tokens - 1) / tokens;
    const double2* vc = a.vc_part + (int64_t)unit * a.vc_stride;
    double Z = 0.0, c_old = 0.0;
    for (int i = threadIdx.x & 63; i < nvc; i += 64) {
      const double2 p = vc[i];
      Z += p.x;
      c_old += p.y;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      Z += __shfl_xor(Z, o);
      c_old += __shfl_xor(c_old, o);
    }
    normalise(Z, c_old);
  }
  // m_used of a position with usage u; its credit is replaced by the new one
  __device__ __forceinline__ float operator()(float u, float& credit) const {
    const float mc = (float)((fmax((double)u, 0.0) + eps) * inv_z);
    float cn = mc, mu = mc;  // lambda == 0: credit not used, the mass passes through unchanged
    if (ema) {
      cn = (float)(lam * (double)credit + (1.0 - lam) * (double)mc);
      mu = (float)(bet * (double)mc + (1.0 - bet) * ((double)cn * inv_csum));
    }
    credit = cn;
    return mu;
  }
};

// A given m_used, four positions per lane: prefixes p inside the piece and the largest of them over the piece (the same in its
// 16 lanes).  A caller's values need not be positive: a threshold may be reached inside a piece whose end lies below it again.
__device__ __forceinline__ double piece_scan(const float (&x)[4], int j0, int T, double (&p)[4]) {
  sub_scan(x, p);
  double top = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (j0 + i < T) top = fmax(top, p[i]);
#pragma unroll
  for (int o = kSubLanes / 2; o >= 1; o >>= 1) top = fmax(top, __shfl_xor(top, o));
  return top;
}

// Split / merge pass over the initial segments, one pass from the left (Alg. 1 step 3, the loop over segments;
// Sec. 3.3 "Mass-based adaptive segmentation").  cut(i), i = 1 .. K, is the end of initial segment i (cut(K) = T).
// A segment longer than l_max becomes ceil(L / l_max) parts whose lengths differ by at most one, the longer ones
// first; one shorter than l_min joins the segment to its left, the very first one stays open so that the next
// initial segment starts where it started; empty initial segments vanish.  Writes the ends of the final segments
// to out[0 .. n) (at most cap of them) and returns n.  A serial chain of at most K steps that the whole first wave
// walks together, its lanes writing the parts of a split side by side (10 us by one lane for 10 -> 133 segments).
template <typename Cut>
__device__ __forceinline__ int split_merge_pass(Cut cut, int K, int T, int l_min, int l_max, int cap, int32_t* out) {
  const int lane = threadIdx.x;
  int n = 0, start = 0;
  bool have_left = false;
  for (int i = 1; i <= K; ++i) {
    const int e = cut(i);
    const int L = e - start;
    if (L == 0) continue;
    if (l_max > 0 && L > l_max) {
      const int parts = (L + l_max - 1) / l_max, base = L / parts, extra = L - base * parts;
      const int fit = min(parts, cap - n);
      for (int j = lane; j < fit; j += 64) out[n + j] = start + (j + 1) * base + min(j + 1, extra);
      n += fit;
      have_left = true;
      start = e;
    } else if (l_min > 0 && L < l_min) {
      if (have_left) {
        if (lane == 0) out[n - 1] = e;
        start = e;
      }
    } else {
      if (n < cap) {
        if (lane == 0) out[n] = e;
        ++n;
      }
      have_left = true;
      start = e;
    }
  }
  if (start < T && n < cap) {  // the whole sequence was one too-short segment
    if (lane == 0) out[n] = T;
    ++n;
  }
  if (n > 0 && lane == 0) out[n - 1] = T;  // (only matters if the capacity cut the list short)
  return n;
}

// The cuts of one unit from the sums of 64 positions, the masses of its segments and its quotas, in one workgroup.
// The prefix over the sums (512 of them for 32768 positions) goes to LDS; every threshold finds its piece there by
// bisection, and 16 lanes scan the 64 positions of that piece for the first one that reaches it.  Only those pieces of
// m_used are read again: latency bounds this kernel, so nothing in it depends on T beyond the prefix, and all thresholds
// travel at once (BLOCK / 16 per round).  6 us for 8 units of 32768 positions and 16 segments, 8 for 256, 9 for 112 of
// 131072 with 32 segments; 23 for 256 units with thresholds k*Delta and 133 final segments (42 with the split / merge pass
// by one lane and the quotas in LDS; with the masses as differences of prefixes, which lose those below 1e-10, 22).
//   CUTS_STEP     fused step: thresholds k/S, at most 64 segments
//   CUTS_GENERAL  fused step: also thresholds k*Delta with the split / merge pass, up to 1024 segments
//   CUTS_STAGE    ams_mass_segment: no quotas, any sign of m_used (the bisection runs over the largest prefix so far)
//   CUTS_OWN      the same without the sums of 64 in memory: the workgroup forms them from m_used, in the same order
//   CUTS_MASS     CUTS_STEP for caches of up to 8 * BLOCK positions, which forms the masses itself (mass_kernel's arithmetic)
//   CUTS_ALL      CUTS_GENERAL for caches of up to 4 * ROUNDS * BLOCK, from the usage alone: pooling, normalisers, masses as well
//   CUTS_UNIT     CUTS_MASS inside the one-launch scorer, on the usage that it holds
enum { CUTS_STEP = 0, CUTS_GENERAL = 1, CUTS_STAGE = 2, CUTS_OWN = 3, CUTS_MASS = 4, CUTS_ALL = 5, CUTS_UNIT = 6 };
constexpr int kStepMaxSeg = 64;

struct CutsOut {
  float* seg_mass;
  int32_t *quota, *idx, *n_kept;
  uint32_t* flags;
  int n_words, budget, q_min, n_sink, n_last;
  const int32_t* status;
  // CUTS_MASS: the usage, the credit (updated in place), where the masses go, and the parameters of Eq. (1) and the EMA
  const float* u;
  float *credit, *m_used;
  float lambda, beta, eps;
};

template <int BLOCK, int KIND, int ROUNDS>
struct CutsLds {
  static constexpr bool kOwn = KIND == CUTS_OWN, kSigned = KIND == CUTS_STAGE || kOwn, kAll = KIND == CUTS_ALL;
  static constexpr bool kMass = KIND == CUTS_MASS || KIND == CUTS_UNIT || kAll;         // forms the masses
  static constexpr bool kStep = KIND == CUTS_STEP || KIND == CUTS_MASS || KIND == CUTS_UNIT;  // thresholds k/S, few of them
  static constexpr int kW = BLOCK / 64, kPerThread = KIND == CUTS_UNIT ? 1 : 4, kCapSub = BLOCK * kPerThread;
  static constexpr int kCap = kStep ? kStepMaxSeg : kMaxSegments;
  __align__(16) float m[KIND == CUTS_UNIT ? 4 : kMass ? BLOCK * 4 * ROUNDS + (kAll ? 2 * kMaxPoolR + 4 : 0) : 4];
  double piece[kAll ? BLOCK * 4 * ROUNDS / kSub : 1];  // the sums of 64, which the prefixes replace
  double ends[kCapSub];                                // prefix at the end of every piece of the group
  double peak[kSigned ? kCapSub : 1];                  // largest prefix up to the end of the piece
  double wave_tot[kW], wave_top[kSigned ? kW : 1];
  double cpre[kCap + 1];
  int32_t bounds[kCap + 1];
  float mass[kCap];
  int32_t reseg[kStep ? 1 : kCap + 1];
  int n_reseg;
};

// CUTS_UNIT: m_sm holds the usage of BLOCK * 4 * ROUNDS positions (the masses take its place), cx the credit of this thread's
// positions, Z and c_old the unit's sums.
template <int BLOCK, int KIND, int ROUNDS>
__device__ __forceinline__ void cuts_body(const MsArgs& a, const float* m_all, const CutsOut& o, int unit, CutsLds<BLOCK, KIND, ROUNDS>& sm,
                                          float* m_sm, float (&cx)[ROUNDS][4], double Z, double c_old) {
  using Lds = CutsLds<BLOCK, KIND, ROUNDS>;
  constexpr int kW = Lds::kW, kPerThread = Lds::kPerThread, kCapSub = Lds::kCapSub, kCap = Lds::kCap, kGroups16 = BLOCK / kSubLanes;
  constexpr bool kOwn = Lds::kOwn, kSigned = Lds::kSigned, kAll = Lds::kAll, kMass = Lds::kMass, kStep = Lds::kStep;
  constexpr bool kUnit = KIND == CUTS_UNIT;
  auto& piece_sm = sm.piece;
  auto& ends = sm.ends;
  auto& peak = sm.peak;
  auto& wave_tot = sm.wave_tot;
  auto& wave_top = sm.wave_top;
  auto& cpre = sm.cpre;
  auto& bounds = sm.bounds;
  auto& mass = sm.mass;
  auto& reseg = sm.reseg;
  auto& n_reseg = sm.n_reseg;
  const int S = a.S;
  const int K = kStep ? S : a.K;  // initial segments: thresholds k = 1 .. K-1
  const bool delta_mode = !kStep && a.delta > 0.0;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const float* m_used = m_all + (int64_t)unit * a.d.t_stride;
  const int n_sub = (T + kSub - 1) / kSub;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = threadIdx.x & (kSubLanes - 1);
  for (int k = threadIdx.x; k <= S; k += BLOCK) {
    bounds[k] = (k == 0) ? 0 : T;
    cpre[k] = (k == 0) ? 0.0 : -1.0;
  }
  double C = 0.0, top = -INFINITY;  // prefix at the end of the groups before, and the largest one so far
#pragma unroll 1
  for (int base = 0; base < n_sub; base += kCapSub) {
    const int n = min(kCapSub, n_sub - base);
    double v[kPerThread], t[kPerThread];
    const int e0 = (int)threadIdx.x * kPerThread;
    if constexpr (kMass) {  // (one group)
      const float* u = o.u + (int64_t)unit * a.d.t_stride;
      float *credit = o.credit + (int64_t)unit * a.d.t_stride, *out = o.m_used + (int64_t)unit * a.d.t_stride;
      float ux[ROUNDS][4];
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const int j0 = (r * BLOCK + (int)threadIdx.x) * 4;
        if constexpr (kUnit) {
          const float4 u4 = *reinterpret_cast<const float4*>(&m_sm[j0]);
          ux[r][0] = u4.x, ux[r][1] = u4.y, ux[r][2] = u4.z, ux[r][3] = u4.w;
        } else {
          load_run(u, j0, T, a.vec, ux[r], 0.f);
          load_run(credit, j0, T, a.vec, cx[r], 0.f);
        }
      }
      if constexpr (kAll) {
        if (a.pool_r > 0) {  // tile[e] = position e - pool_r
          for (int e = threadIdx.x; e < a.pool_r; e += BLOCK) {
            m_sm[e] = 0.f;
            m_sm[BLOCK * 4 * ROUNDS + a.pool_r + e] = 0.f;
          }
#pragma unroll
          for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) m_sm[(r * BLOCK + (int)threadIdx.x) * 4 + i + a.pool_r] = ux[r][i];  // (0 past the end)
          __syncthreads();
#pragma unroll
          for (int r = 0; r < ROUNDS; ++r) {
            const int j0 = (r * BLOCK + (int)threadIdx.x) * 4;
            pool_run(m_sm, j0, j0, T, a.pool_r, ux[r]);
          }
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((r * BLOCK + (int)threadIdx.x) * 4 + i < T) {
              Z += fmax((double)ux[r][i], 0.0) + (double)o.eps;
              c_old += (double)cx[r][i];
            }
        Z = block_sum<kW>(Z, wave_tot);
        c_old = block_sum<kW>(c_old, wave_tot);
        __syncthreads();  // wave_tot and the tile are written again
      }
      const MassOf mass = kAll || kUnit ? MassOf(o.lambda, o.beta, o.eps, Z, c_old) : MassOf(a, unit, T, o.lambda, o.beta, o.eps);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const int j0 = (r * BLOCK + (int)threadIdx.x) * 4;
        float mu[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mu[i] = j0 + i < T ? mass(ux[r][i], cx[r][i]) : 0.f;
        *reinterpret_cast<float4*>(&m_sm[j0]) = make_float4(mu[0], mu[1], mu[2], mu[3]);
        double p[4];
        sub_scan(mu, p);
        if (l16 == kSubLanes - 1 && j0 - (kSub - 4) < T) {
          ends[j0 / kSub] = p[3];
          if (kAll) piece_sm[j0 / kSub] = p[3];
        }
        store_run(credit, j0, T, a.vec, cx[r]);
        store_run(out, j0, T, a.vec, mu);
      }
      __syncthreads();
    }
    if constexpr (kOwn) {
      for (int first = 0; first < n; first += 4 * kGroups16) {  // four pieces per 16 lanes in flight
        const int e = first + (int)threadIdx.x / kSubLanes;
        float x[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) load_run(m_used, (base + e + r * kGroups16) * kSub + l16 * 4, T, a.vec, x[r], 0.f);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double p[4];
          const double t16 = piece_scan(x[r], (base + e + r * kGroups16) * kSub + l16 * 4, T, p);
          if (l16 == kSubLanes - 1 && e + r * kGroups16 < n) ends[e + r * kGroups16] = p[3], peak[e + r * kGroups16] = t16;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      v[i] = 0.0;
      t[i] = -INFINITY;
      if (e0 + i < n) {
        const int64_t at = (int64_t)unit * a.n_sub + base + e0 + i;
        if (kMass) {  // this thread's four entries, which it replaces by the prefixes below
          v[i] = ends[e0 + i];
        } else if (kOwn) {
          v[i] = ends[e0 + i];
          t[i] = peak[e0 + i];
        } else if (kSigned) {
          const double2 p = ((const double2*)a.sub)[at];
          v[i] = p.x;
          t[i] = p.y;
        } else {
          v[i] = a.sub[at];
        }
      }
    }
    double ts = v[0];
#pragma unroll
    for (int i = 1; i < kPerThread; ++i) ts += v[i];
    double incl = ts;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const double x = __shfl_up(incl, d);
      if (lane >= d) incl += x;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    double run = C;
    for (int w = 0; w < wave; ++w) run += wave_tot[w];
    run += incl - ts;
    double local_top = -INFINITY;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      t[i] += run;  // the piece's prefixes start where the one before it ends
      local_top = fmax(local_top, t[i]);
      t[i] = local_top;
      run += v[i];
      ends[e0 + i] = run;
    }
    if (kSigned) {
      double it = local_top;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const double x = __shfl_up(it, d);
        if (lane >= d) it = fmax(it, x);
      }
      double before = __shfl_up(it, 1);
      if (lane == 0) before = -INFINITY;
      if (lane == 63) wave_top[wave] = it;
      __syncthreads();
      before = fmax(before, top);
      for (int w = 0; w < wave; ++w) before = fmax(before, wave_top[w]);
#pragma unroll
      for (int i = 0; i < kPerThread; ++i) peak[e0 + i] = fmax(before, t[i]);
    }
    __syncthreads();
    const double* reach = kSigned ? peak : ends;  // never falls (up to a NaN, which ends the search)
    const double C_end = ends[n - 1], reach0 = kSigned ? top : C, reach1 = reach[n - 1];
    for (int k = 1 + (int)threadIdx.x / kSubLanes; k < K; k += kGroups16) {
      const double thr = delta_mode ? (double)k * a.delta : (double)k / (double)S;
      if (!(thr > reach0) || reach1 < thr) continue;  // in an earlier group, or not in this one
      int lo = 0, hi = n - 1;  // first piece whose end does not lie below the threshold
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (reach[mid] < thr)
          lo = mid + 1;
        else
          hi = mid;
      }
      const int j0 = (base + lo) * kSub + l16 * 4;
      float x[4];
      if constexpr (kMass) {
        const float4 x4 = *reinterpret_cast<const float4*>(&m_sm[j0]);
        x[0] = x4.x, x[1] = x4.y, x[2] = x4.z, x[3] = x4.w;
      } else {
        load_run(m_used, j0, T, a.vec, x, 0.f);
      }
      double p[4];
      sub_scan(x, p);
      const double before = lo > 0 ? ends[lo - 1] : C;
      int j = INT32_MAX;  // first position of this lane that reaches the threshold
      double P = 0.0;
#pragma unroll
      for (int i = 3; i >= 0; --i)
        if (j0 + i < T && before + p[i] >= thr) {
          j = j0 + i;
          P = before + p[i];
        }
      const uint64_t reached = __ballot(j != INT32_MAX) >> (lane & ~(kSubLanes - 1)) & ((1u << kSubLanes) - 1);
      if (reached) {
        if (l16 == __ffsll((long long)reached) - 1) {
          bounds[k] = j + 1;
          cpre[k] = P;
        }
      } else if (reach[lo] >= thr) {  // only the rounding of the start of the piece lies in between: where it is highest
        P = -INFINITY;
#pragma unroll
        for (int i = 3; i >= 0; --i)
          if (j0 + i < T && before + p[i] >= P) {
            j = j0 + i;
            P = before + p[i];
          }
#pragma unroll
        for (int d = 1; d < kSubLanes; d <<= 1) {
          const double P2 = __shfl_xor(P, d);
          const int j2 = __shfl_xor(j, d);
          if (P2 > P || (P2 == P && j2 < j)) {
            P = P2;
            j = j2;
          }
        }
        if (l16 == 0) {
          bounds[k] = j + 1;
          cpre[k] = P;
        }
      }
    }
    C = C_end;
    top = reach1;
    if (base + kCapSub < n_sub) __syncthreads();  // the next group overwrites what the searches read
    if (kOwn && delta_mode && n_sub <= kCapSub) {  // the sums of 64 once more, for the masses below
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kPerThread; ++i) peak[e0 + i] = v[i];
    }
  }
  __syncthreads();
  const double total = C;
  if (delta_mode) {
    if (wave == 0) {
      const int n = split_merge_pass([&](int i) { return i == K ? T : bounds[i]; }, K, T, a.l_min, a.l_max, S, reseg);
      if (lane == 0) n_reseg = n;
    }
    __syncthreads();
    const int n = n_reseg;
    for (int i = threadIdx.x; i < S; i += BLOCK) bounds[i + 1] = i < n ? reseg[i] : T;
    __syncthreads();
    // the masses of the final segments: each the sum of its own positions (the whole pieces inside and the rest of the
    // pieces at its ends), because a segment may hold far less than the last bit of the prefix in front of it
    for (int sg = (int)threadIdx.x / kSubLanes; sg < S; sg += kGroups16) {
      const int lo = bounds[sg], hi = bounds[sg + 1], q0 = lo / kSub, q1 = (hi - 1) / kSub;
      double sum = 0.0;
      if (hi > lo) {
        const int t0 = q0 * kSub + l16 * 4, t1 = q1 * kSub + l16 * 4;
        float x0[4], x1[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (kMass) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            x0[i] = t0 + i < hi ? m_sm[t0 + i] : 0.f;
            if (q1 > q0 && t1 + i < hi) x1[i] = m_sm[t1 + i];
          }
        } else {
          load_run(m_used, t0, hi, a.vec, x0, 0.f);
          if (q1 > q0) load_run(m_used, t1, hi, a.vec, x1, 0.f);
        }
        if (kOwn && n_sub > kCapSub) {
          for (int q = q0 + 1; q < q1; q += 4) {
            float x[4][4];
#pragma unroll
            for (int r = 0; r < 4; ++r) load_run(m_used, (q + r) * kSub + l16 * 4, q1 * kSub, a.vec, x[r], 0.f);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              double p[4];
              sub_scan(x[r], p);
              const double v = __shfl(p[3], lane | (kSubLanes - 1));
              if (q + r < q1 && ((q + r - q0 - 1) & (kSubLanes - 1)) == l16) sum += v;
            }
          }
        } else {
#pragma unroll 4
          for (int q = q0 + 1 + l16; q < q1; q += kSubLanes) {
            const int64_t at = (int64_t)unit * a.n_sub + q;
            sum += kAll ? piece_sm[q] : kOwn ? peak[q] : kSigned ? ((const double2*)a.sub)[at].x : a.sub[at];
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) sum += (t0 + i >= lo ? (double)x0[i] : 0.0) + (double)x1[i];
      }
#pragma unroll
      for (int d = kSubLanes / 2; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
      if (l16 == 0) mass[sg] = (float)sum;
    }
  } else {
    for (int i = threadIdx.x; i < S; i += BLOCK) {
      const double lo = cpre[i] < 0.0 ? total : cpre[i];
      const double hi = (i + 1 == S || cpre[i + 1] < 0.0) ? total : cpre[i + 1];
      mass[i] = (float)(hi - lo);
    }
  }
  __syncthreads();
  if (o.seg_mass)
    for (int i = threadIdx.x; i < S; i += BLOCK) o.seg_mass[(int64_t)unit * S + i] = mass[i];
  for (int i = threadIdx.x; i <= S; i += BLOCK) a.bounds[(int64_t)unit * (S + 1) + i] = bounds[i];
  if constexpr (!kSigned) {
    // what the quota kernels do besides the quotas: the -1 tail of idx, the kept count, the cleared bitmap
    // of the must-keep path; sinks and the recent suffix come out of the budget first
    const int kept = min(o.budget, T);
    const int sinks = min(o.n_sink, kept);
    const int bud = kept - sinks - min(o.n_last, kept - sinks);
    int32_t* idx = o.idx + (int64_t)unit * o.budget;
    for (int j = kept + threadIdx.x; j < o.budget; j += BLOCK) idx[j] = -1;
    // a scorer whose bounded wait expired left unfinished scores: no unit reports a kept set then
    if (threadIdx.x == 0) o.n_kept[unit] = (o.status && *o.status != 0) ? -1 : kept;
    if (o.flags)
      for (int j = threadIdx.x; j < o.n_words; j += BLOCK) o.flags[(int64_t)unit * o.n_words + j] = 0u;
    if (threadIdx.x < 64) quota_store<kCap>(S, bud, o.q_min, bounds, mass, o.quota + (int64_t)unit * S);
  }
}

// The arguments of a fused step's cuts.
struct UnitCuts {
  MsArgs a;
  CutsOut o;
};

}  // namespace ams
#endif
