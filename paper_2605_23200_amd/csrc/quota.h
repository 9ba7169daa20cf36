// Quota of every segment of one unit by one wave (Sec. 3.3 "Segment-wise Quota Allocation"; Alg. 1 step 4).
// Shared by the stand-alone quota kernel and the per-unit kernel of the fused step.
#ifndef AMS_QUOTA_H
#define AMS_QUOTA_H

#include <type_traits>

#include "ams_internal.h"

namespace ams {

// Sum over the wave, the same value in every lane: the rows of 16 lanes by DPP, the four rows by scalar reads.
__device__ __forceinline__ int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);  // row_ror:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true);
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
         (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}

// Value of lane j, the same j in every lane: two scalar reads instead of a trip through the LDS crossbar.
__device__ __forceinline__ double lane_f64(double v, int j) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, j);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), j);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Quotas of up to 64 * R segments by one wave: lane i owns the segments i, i + 64, ...; quo[r] is the quota of segment
// 64 r + lane.  bounds and mass lie in LDS.  Sums of masses run in index order over the open segments and every share is
// rem * M_i / sum, the same operations in the same order as plain C.  A serial chain: sums and counts travel through
// scalar lane reads and ballots, and the leftovers go to the largest fractions by bisection on their bit patterns, not
// by comparing every pair.  With R = 16 the lane reads want more scalar registers than there are: 683 of them live in lanes of
// vector registers (no memory is touched), 3 us for 139 segments.
template <int R>
__device__ __forceinline__ void quota_wave(int S, int bud, int q_min, const int32_t* bounds, const float* mass,
                                           int (&quo)[R]) {
  const int lane = threadIdx.x;
  auto len = [&](int r) __attribute__((always_inline)) {
    const int i = r * 64 + lane;
    return i < S ? bounds[i + 1] - bounds[i] : 0;
  };
  int c_nonempty = 0, c_need = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    c_nonempty += __popcll(__ballot(len(r) > 0));
    c_need += min(q_min, len(r));
  }
  int floor_q = q_min;
  if (wave_sum(c_need) > bud) floor_q = c_nonempty > 0 ? bud / c_nonempty : 0;
  double raw[R];
  bool active[R];
  int c_lo = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int n = len(r);
    quo[r] = min(floor_q, n);
    active[r] = n > quo[r];
    raw[r] = 0.0;
    c_lo += quo[r];
  }
  int rem = bud - wave_sum(c_lo);
  // proportional shares; a segment whose share reaches its room is filled and leaves the pool
  for (;;) {
    int n_active = 0;
    double msum = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) n_active += __popcll(__ballot(active[r]));
    if (n_active == 0 || rem <= 0) break;
#pragma unroll
    for (int r = 0; r < R; ++r) {  // index order; a closed segment adds an exact zero
      const double open = active[r] ? (double)mass[r * 64 + lane] : 0.0;
#pragma unroll
      for (int j0 = 0; j0 < 64; j0 += 16)
        if (r * 64 + j0 < S) {
#pragma unroll
          for (int j = j0; j < j0 + 16; ++j) msum += lane_f64(open, j);
        }
    }
    int c_taken = 0;
    bool any_sat = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      bool sat = false;
      if (active[r]) {
        const int n = len(r), room = n - quo[r];
        raw[r] = msum > 0.0 ? (double)rem * (double)mass[r * 64 + lane] / msum : (double)rem / (double)n_active;
        sat = raw[r] >= (double)room;
        if (sat) {
          quo[r] = n;
          active[r] = false;
          c_taken += room;
        }
      }
      any_sat = any_sat || __ballot(sat) != 0;
    }
    if (!any_sat) break;
    rem -= wave_sum(c_taken);
  }
  if (rem > 0) {
    // a fraction lies in [0, 1): its bit pattern orders like the number
    uint64_t key[R];
    int c_given = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool real = active[r] && raw[r] == raw[r];  // masses that are no numbers: everybody ranks alike
      const double fl = real ? floor(raw[r]) : 0.0;
      key[r] = real ? __builtin_bit_cast(uint64_t, raw[r] - fl) : 0;
      quo[r] += (int)fl;
      c_given += (int)fl;
    }
    int left = rem - wave_sum(c_given);
    // one extra each, largest fractional part first, equal parts by lower segment index
    while (left > 0) {
      bool can[R];
      int n_can = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        can[r] = active[r] && quo[r] < len(r);
        n_can += __popcll(__ballot(can[r]));
      }
      if (n_can == 0) break;
      if (n_can <= left) {
#pragma unroll
        for (int r = 0; r < R; ++r) quo[r] += can[r] ? 1 : 0;
        left -= n_can;
        continue;
      }
      // the left-th largest fraction, bit by bit from the top, until a bound separates exactly `left` of them
      auto at_least = [&](uint64_t c) __attribute__((always_inline)) {
        int n = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) n += __popcll(__ballot(can[r] && key[r] >= c));
        return n;
      };
      constexpr uint64_t kHalf = 0x3FE0000000000000ull;  // 0.5: all fractions from there on share the upper bits
      uint64_t thr = 0;
      int bit = 61, n_thr = n_can;
      if (const int n = at_least(kHalf); n >= left) {
        thr = kHalf;
        n_thr = n;
        bit = 51;
      }
      for (; bit >= 0 && n_thr != left; --bit) {
        const uint64_t c = thr | (1ull << bit);
        if (const int n = at_least(c); n >= left) {
          thr = c;
          n_thr = n;
        }
      }
      // more than `left` reach the bound only if they are equal to it: of those the lower segments are served
      int spare = n_thr - left, n_eq = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) n_eq += __popcll(__ballot(can[r] && key[r] == thr));
      int keep_eq = n_eq - spare;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint64_t eq = __ballot(can[r] && key[r] == thr);
        const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        const bool take = can[r] && (key[r] > thr || (key[r] == thr && (int)__popcll(eq & below) < keep_eq));
        quo[r] += take ? 1 : 0;
        keep_eq -= (int)__popcll(eq);
      }
      left = 0;
    }
  }
}

// The quotas of S <= MAX_S segments -> out[0 .. S), by the first wave of the workgroup.
template <int MAX_S>
__device__ __forceinline__ void quota_store(int S, int bud, int q_min, const int32_t* bounds, const float* mass,
                                            int32_t* out) {
  auto run = [&](auto r_c) __attribute__((always_inline)) {
    constexpr int R = decltype(r_c)::value;
    int quo[R];
    quota_wave<R>(S, bud, q_min, bounds, mass, quo);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r * 64 + (int)threadIdx.x < S) out[r * 64 + threadIdx.x] = quo[r];
  };
  if (MAX_S <= 64 || S <= 64) return run(std::integral_constant<int, 1>{});
  if constexpr (MAX_S > 64) {
    if (S <= 256) return run(std::integral_constant<int, 4>{});
    run(std::integral_constant<int, 16>{});
  }
}

}  // namespace ams
#endif
