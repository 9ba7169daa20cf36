// Segment quotas, in-segment top-k and the kept set (Sec. 3.3 "Segment-wise Quota Allocation",
// "In-Segment Selection" and the must-keep rules; Alg. 1 steps 4-5).
//
// quota_kernel   one wave per unit, the segments in registers; the
//                arithmetic is a handful of double operations per segment and is done in index
//                order so that it is reproducible bit for bit.
// select_kernel  one workgroup per (segment, unit): the quota-th largest score on an order-preserving integer
//                image of the floats, then an ordered compaction that keeps everything above the
//                threshold and the first few positions equal to it, ascending.  In the fused step it
//                may gather the kept rows too (Alg. 1 step 6), several workgroups to a segment where
//                the launch is small.
// finalize_kernel  (only with a must-keep set) one workgroup per unit.  The segment picks arrive as
//                bits of a per-unit bitmap, so the union with the must-keep positions and the removal
//                of duplicates are one OR; what the duplicates leave open is filled with the best
//                scores outside the set (the same selection over the unset positions, from memory where the
//                sequence is too long for registers), and the ascending index list is read off the bitmap.
#include "ams_internal.h"
#include "quota.h"

namespace ams {
namespace {

constexpr int kMaxSeg = 1024;

// What the quota kernel does before the quotas: the -1 tail of idx, the kept count, the cleared bitmap of the
// must-keep path.  Returns the budget the segments share.
__device__ __forceinline__ int quota_prologue(const Dims& d, const int32_t* seq_lens, int budget,
                                              int32_t* idx_all, int32_t* n_kept_all, int n_sink, int n_last,
                                              uint32_t* flags_all, int n_words) {
  const int unit = blockIdx.x, nthr = blockDim.x;
  int l, b, h;
  unit_coords(d, unit, l, b, h);
  const int T = seq_len(d, seq_lens, b);
  // must-keep positions go in first: sinks always, the recent suffix as far as it fits; the segments
  // share what is left
  const int kept = min(budget, T);
  const int sinks = min(n_sink, kept);
  const int bud = kept - sinks - min(n_last, kept - sinks);
  int32_t* idx = idx_all + (int64_t)unit * budget;
  // entries of idx beyond the kept count are -1
  for (int j = kept + threadIdx.x; j < budget; j += nthr) idx[j] = -1;
  if (threadIdx.x == 0) n_kept_all[unit] = kept;
  if (flags_all)
    for (int j = threadIdx.x; j < n_words; j += nthr) flags_all[(int64_t)unit * n_words + j] = 0u;
  return bud;
}

__global__ __launch_bounds__(64) void quota_kernel(Dims d, const int32_t* seq_lens, int S, int budget,
                                                   int q_min, const int32_t* bounds_all,
                                                   const float* seg_mass_all, int32_t* quota_all,
                                                   int32_t* idx_all, int32_t* n_kept_all, int n_sink, int n_last,
                                                   uint32_t* flags_all, int n_words) {
  __shared__ int32_t bounds[kMaxSeg + 1];
  __shared__ float mass[kMaxSeg];
  const int unit = blockIdx.x;
  for (int i = threadIdx.x; i < S; i += 64) {
    bounds[i] = bounds_all[(int64_t)unit * (S + 1) + i];
    mass[i] = seg_mass_all[(int64_t)unit * S + i];
  }
  if (threadIdx.x == 0) bounds[S] = bounds_all[(int64_t)unit * (S + 1) + S];
  const int bud = quota_prologue(d, seq_lens, budget, idx_all, n_kept_all, n_sink, n_last, flags_all, n_words);
  __syncthreads();
  quota_store<kMaxSeg>(S, bud, q_min, bounds, mass, quota_all + (int64_t)unit * S);
}

// Order-preserving image of a score: larger float <-> larger unsigned; -0 and +0 coincide and
// NaN ranks with -infinity.
__device__ __forceinline__ uint32_t score_key(float x) {
  if (x != x) x = -INFINITY;
  if (x == 0.f) x = 0.f;
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Where a selected position goes: slot `slot` of the ascending index list (if it lies in the workgroup's share [r0, r1)),
// or its bit of the bitmap.
template <bool FLAGS>
struct Emit {
  int32_t* out;
  uint32_t* flags;
  int r0, r1;
  __device__ __forceinline__ void operator()(int slot, int t) const {
    if (FLAGS)
      atomicOr(&flags[t >> 5], 1u << (t & 31));
    else if (slot >= r0 && slot < r1)
      out[slot] = t;
  }
};

// What a selection workgroup does with its picks: index list, bits of the unit's map, or index list and gather.
enum { SELECT_LIST = 0, SELECT_FLAGS = 1, SELECT_GATHER = 2 };
constexpr int kGatherLongest = 2560;  // expected length of a segment up to which its workgroup gathers as well
constexpr int kGatherList = 512;  // picks kept in LDS for the gather; later ones are read back from the index list

struct GatherArgs {
  KvDev ks, vs, kd, vd;
  const float* credit_src;
  float* credit_dst;
  const int32_t* n_kept;
  int budget, parts;
};

// The kept rows of one segment, picks [r0, r1) of it (pick j sits in row out0 + j of the compacted cache): K' = K[idx],
// V' = V[idx] and the credit (Alg. 1 step 6; App. E for a paged destination).
template <int BLOCK, typename Pos>
__device__ __forceinline__ void gather_rows(const Dims& d, const GatherArgs& ga, int unit, int out0, int r0, int r1, Pos pos) {
  int l, b, h;
  unit_coords(d, unit, l, b, h);
  const int lanes = ga.ks.row_bytes / 16, per = BLOCK / lanes;
  const int sub = threadIdx.x % lanes, r = threadIdx.x / lanes;
  const float* c_src = ga.credit_src + (int64_t)unit * d.t_stride;
  float* c_dst = ga.credit_dst ? ga.credit_dst + (int64_t)unit * ga.budget + out0 : nullptr;
  int jc = r0 + (int)threadIdx.x;
  float c = 0.f;  // travels with the first rows
  if (c_dst && jc < r1) c = c_src[pos(jc)];
  for (int j = r0 + r; j < r1; j += 2 * per) {
    const bool two = j + per < r1;
    const int t0 = pos(j), t1 = two ? pos(j + per) : t0;
    const uint4 k0 = *(const uint4*)(kv_row(ga.ks, l, b, h, t0) + sub * 16);
    const uint4 v0 = *(const uint4*)(kv_row(ga.vs, l, b, h, t0) + sub * 16);
    const uint4 k1 = *(const uint4*)(kv_row(ga.ks, l, b, h, t1) + sub * 16);
    const uint4 v1 = *(const uint4*)(kv_row(ga.vs, l, b, h, t1) + sub * 16);
    *(uint4*)(kv_row(ga.kd, l, b, h, out0 + j) + sub * 16) = k0;
    *(uint4*)(kv_row(ga.vd, l, b, h, out0 + j) + sub * 16) = v0;
    if (two) {
      *(uint4*)(kv_row(ga.kd, l, b, h, out0 + j + per) + sub * 16) = k1;
      *(uint4*)(kv_row(ga.vd, l, b, h, out0 + j + per) + sub * 16) = v1;
    }
  }
  if (c_dst && jc < r1) {
    c_dst[jc] = c;
    for (jc += BLOCK; jc < r1; jc += BLOCK) c_dst[jc] = c_src[pos(jc)];
  }
}

// The selection kernel holds the keys of a segment in registers: BLOCK threads with PER keys each.  One wave takes the
// many short segments (no barriers between waves), 256, 512 and 1024 threads the longer ones; a segment that is longer
// than its shape's BLOCK * PER is selected from memory.

// Inclusive sum over the lanes of a wave (DPP: inside the rows of 16, then the rows' ends into the rows after them).
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Lowest and highest key of the wave, the same in every lane.
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi) {
#define AMS_ROR(X, CTRL) (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(X), CTRL, 0xf, 0xf, true)
  lo = min(lo, AMS_ROR(lo, 0x128)), hi = max(hi, AMS_ROR(hi, 0x128));
  lo = min(lo, AMS_ROR(lo, 0x124)), hi = max(hi, AMS_ROR(hi, 0x124));
  lo = min(lo, AMS_ROR(lo, 0x122)), hi = max(hi, AMS_ROR(hi, 0x122));
  lo = min(lo, AMS_ROR(lo, 0x121)), hi = max(hi, AMS_ROR(hi, 0x121));
#undef AMS_ROR
  uint32_t l = 0xFFFFFFFFu, h = 0;
#pragma unroll
  for (int r = 0; r < 64; r += 16) {
    l = min(l, (uint32_t)__builtin_amdgcn_readlane((int)lo, r));
    h = max(h, (uint32_t)__builtin_amdgcn_readlane((int)hi, r));
  }
  lo = l;
  hi = h;
}

// Of 256 bins over the keys from lo on, 2^sh keys wide: the one in which the count from the top reaches rem, found by every
// wave for itself, lane 0 the highest bins.  lo and rem move on to that bin, n_bin is what it holds.
__device__ __forceinline__ void top_bin(const int* h, int lane, int& rem, uint32_t& lo, int sh, int& n_bin) {
  const int4 c = *reinterpret_cast<const int4*>(&h[252 - 4 * lane]);
  const int s = (c.x + c.y) + (c.z + c.w);
  const int above = wave_scan(s) - s;
  const bool mine = above < rem && rem <= above + s;
  const int c3 = above + c.w, c2 = c3 + c.z, c1 = c2 + c.y;
  int bin = 252 - 4 * lane, cum = c1, in = c.x;
  if (rem <= c3) {
    bin += 3, cum = above, in = c.w;
  } else if (rem <= c2) {
    bin += 2, cum = c3, in = c.z;
  } else if (rem <= c1) {
    bin += 1, cum = c2, in = c.y;
  }
  const int src = __ffsll((long long)__ballot(mine)) - 1;
  bin = __builtin_amdgcn_readlane(bin, src);
  rem -= __builtin_amdgcn_readlane(cum, src);
  n_bin = __builtin_amdgcn_readlane(in, src);
  lo += (uint32_t)bin << sh;
}

// ---- Segments longer than the registers hold: the scores are read from memory in every pass ----
// Bound: one CU reads the scores four times, six or seven at most, and adds keys to their bins in LDS in one of these passes or a few.
// The range of the keys; bins over it until the bin with the last pick holds few keys (1024 threads: 2048 bins, one to three
// passes; fewer threads: 256 bins, up to four); those keys into LDS, where the bins are refined down to one key (or, where the
// bin is taken as a whole or its keys are equal, a count of the picks of every stretch); the picks in ascending order.  Every wave reads a stretch of its own with 16-byte loads, so that its
// counts place its picks and no pass has a barrier inside.  A unit in one segment: 72 us for 32 units of 74913 scores (181 with
// four radix passes of 4-byte loads and two barriers per 1024 positions of the last one), 42 for 16 of 40000 (98).
template <int BLOCK>
struct FarLds {
  static constexpr int kW = BLOCK / 64, kLogBins = BLOCK == 1024 ? 11 : 8, kBins = 1 << kLogBins;
  static constexpr int kKeys = BLOCK == 1024 ? 1024 : 64;  // at most one per thread
  int bins[kBins + kBins / 32];  // a word of padding per 32: a lane sums up neighbouring bins
  uint2 key[kKeys];              // (key, wave that reads its position)
  uint2 red[kW];
  int above[kW], equal[kW];      // picks of a wave's stretch above the threshold, keys equal to it
  int n_keys;
};

template <int BLOCK>
union BinsOrFar {
  int hist[2][256];  // keys in registers: the bins of two passes
  FarLds<BLOCK> far;
};

// Calls f(t, k, kept) for this wave's stretch of [a, b), four positions t .. t + 3 per lane; load(t, k) gives their keys (0: not
// to be considered) and returns the mask of positions that are kept whatever their key.
template <int BLOCK, typename Load, typename F>
__device__ __forceinline__ void far_walk(int a, int b, Load load, F f) {
  constexpr int kW = BLOCK / 64, kAhead = BLOCK == 1024 ? 6 : 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int first = a & ~255, groups = (b - first + 255) >> 8;
  const int g0 = groups * wave / kW, g1 = groups * (wave + 1) / kW;
  for (int g = g0; g < g1; g += kAhead) {
    uint32_t k[kAhead][4], kept[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      kept[i] = k[i][0] = k[i][1] = k[i][2] = k[i][3] = 0;
      if (g + i < g1) kept[i] = load(first + (g + i) * 256 + lane * 4, k[i]);
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (g + i < g1) f(first + (g + i) * 256 + lane * 4, k[i], kept[i]);
  }
}

// The scores at t .. t + 3 that lie in [a, b), t a multiple of 4; vec: 16-byte reads are aligned and stay in the row.
__device__ __forceinline__ void far_scores(const float* g, int a, int b, int t, bool vec, uint32_t (&k)[4]) {
  float x[4] = {0.f, 0.f, 0.f, 0.f};
  if (t + 3 >= a && t < b) {
    if (vec) {
      const float4 v = *reinterpret_cast<const float4*>(g + t);
      x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (t + i >= a && t + i < b) x[i] = g[t + i];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) k[i] = t + i >= a && t + i < b ? score_key(x[i]) : 0u;  // no score has the key 0
}

// See top_bin; the bins of a FarLds.
template <int BLOCK>
__device__ __forceinline__ void far_top_bin(const FarLds<BLOCK>& s, int& rem, uint32_t& lo, int sh, int& n_bin) {
  constexpr int kPer = FarLds<BLOCK>::kBins / 64;
  const int lane = threadIdx.x & 63, b0 = kPer * (63 - lane);  // lane 0 the highest bins
  int c[kPer], t = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    c[i] = s.bins[b0 + i + (b0 + i) / 32];
    t += c[i];
  }
  const int front = wave_scan(t) - t;
  int bin = b0, cum = front, in = 0, run = front;
  bool open = true;
#pragma unroll
  for (int i = kPer - 1; i >= 0; --i) {
    if (open && rem <= run + c[i]) {
      open = false;
      bin = b0 + i, cum = run, in = c[i];
    }
    run += c[i];
  }
  const int src = __ffsll((long long)__ballot(front < rem && rem <= front + t)) - 1;
  bin = __builtin_amdgcn_readlane(bin, src);
  rem -= __builtin_amdgcn_readlane(cum, src);
  n_bin = __builtin_amdgcn_readlane(in, src);
  lo += (uint32_t)bin << sh;
}

// The q best keys of [a, b) (load: see far_walk; 1 <= q, fewer than there are keys to consider) and the positions kept whatever
// their key, in ascending order: emit(slot, t).  any = false: those positions alone.
template <int BLOCK, typename Load, typename Emit>
__device__ __forceinline__ void far_select(FarLds<BLOCK>& s, int a, int b, int q, bool any, Load load, Emit emit) {
  using F = FarLds<BLOCK>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto clear = [&]() __attribute__((always_inline)) {
    for (int i = threadIdx.x; i < F::kBins + F::kBins / 32; i += BLOCK) s.bins[i] = 0;
  };
  clear();
  if (threadIdx.x == 0) s.n_keys = 0;
  uint32_t thr = 0xFFFFFFFFu;  // keys above it are picked, and the first rem equal to it
  int rem = 0;
  bool counted = false;
  if (any) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    far_walk<BLOCK>(a, b, load, [&](int, const uint32_t (&k)[4], uint32_t) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k[i]) lo = min(lo, k[i]);
        hi = max(hi, k[i]);
      }
    });
    wave_min_max(lo, hi);
    if (lane == 0) s.red[wave] = make_uint2(lo, hi);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < F::kW; ++w) {
      lo = min(lo, s.red[w].x);
      hi = max(hi, s.red[w].y);
    }
    int sh = max(0, 32 - F::kLogBins - (int)__clz((int)((hi - lo) | 1u))), n_bin = 0;
    uint32_t span = hi - lo;  // see select_kernel
    auto add = [&](uint32_t k) __attribute__((always_inline)) {
      const uint32_t off = k - lo;
      if (k >= lo && off <= span) atomicAdd(&s.bins[(off >> sh) + (off >> sh) / 32], 1);
    };
    auto narrow = [&]() __attribute__((always_inline)) {
      __syncthreads();
      far_top_bin<BLOCK>(s, rem, lo, sh, n_bin);
      span = (1u << sh) - 1u;
    };
    auto finer = [&]() __attribute__((always_inline)) {
      sh = max(0, sh - F::kLogBins);
      __syncthreads();
      clear();
      __syncthreads();
    };
    rem = q;
    for (;;) {
      far_walk<BLOCK>(a, b, load, [&](int, const uint32_t (&k)[4], uint32_t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) add(k[i]);  // (lo is above 0)
      });
      narrow();
      if (n_bin <= F::kKeys || n_bin == rem || sh == 0) break;
      finer();
    }
    if (n_bin != rem && n_bin <= F::kKeys) {  // the rest among the bin's keys, in LDS
      int above = 0;
      far_walk<BLOCK>(a, b, load, [&](int, const uint32_t (&k)[4], uint32_t kept) __attribute__((always_inline)) {
        above += __popc(kept);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (k[i] < lo) continue;
          if (k[i] - lo > span)
            ++above;
          else
            s.key[atomicAdd(&s.n_keys, 1)] = make_uint2(k[i], (uint32_t)wave);
        }
      });
      above = wave_sum(above);
      if (lane == 0) {
        s.above[wave] = above;
        s.equal[wave] = 0;
      }
      __syncthreads();
      const int n = s.n_keys;
      const uint2 mine = (int)threadIdx.x < n ? s.key[threadIdx.x] : make_uint2(0u, 0u);
      while (n_bin != rem && sh > 0) {
        finer();
        add(mine.x);
        narrow();
      }
      thr = lo;
      if (n_bin == rem) thr = lo - 1, rem = 0;
      if (mine.x > thr) atomicAdd(&s.above[mine.y], 1);
      if (mine.x == thr) atomicAdd(&s.equal[mine.y], 1);
      counted = true;
    } else {  // the bin as a whole, or its keys are equal
      thr = lo;
      if (n_bin == rem) thr = lo - 1, rem = 0;
    }
  }
  if (!counted) {
    int above = 0, equal = 0;
    far_walk<BLOCK>(a, b, load, [&](int, const uint32_t (&k)[4], uint32_t kept) __attribute__((always_inline)) {
      above += __popc(kept);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        above += k[i] > thr;
        equal += k[i] == thr;
      }
    });
    above = wave_sum(above);
    equal = wave_sum(equal);
    if (lane == 0) {
      s.above[wave] = above;
      s.equal[wave] = equal;
    }
  }
  __syncthreads();
  int n_gt = 0, n_eq = 0;  // in front of this wave's stretch
  for (int w = 0; w < wave; ++w) {
    n_gt += s.above[w];
    n_eq += s.equal[w];
  }
  far_walk<BLOCK>(a, b, load, [&](int t, const uint32_t (&k)[4], uint32_t kept) __attribute__((always_inline)) {
    uint32_t gt = kept, eq = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      gt |= (k[i] > thr ? 1u : 0u) << i;
      eq |= (k[i] == thr ? 1u : 0u) << i;
    }
    const int c = __popc(gt) | __popc(eq) << 16;
    const int incl = wave_scan(c), before = incl - c, all = __builtin_amdgcn_readlane(incl, 63);
    int gt_in_front = n_gt + (before & 0xFFFF), eq_in_front = n_eq + (before >> 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool is_gt = (gt >> i) & 1u, is_eq = (eq >> i) & 1u;
      if (is_gt || (is_eq && eq_in_front < rem)) emit(gt_in_front + min(eq_in_front, rem), t + i);
      gt_in_front += is_gt;
      eq_in_front += is_eq;
    }
    n_gt += all & 0xFFFF;
    n_eq += all >> 16;
  });
}

// The q largest keys of a segment.  Latency and LDS atomics bound this kernel (a few thousand keys per workgroup), so the
// steps that need all threads are few: the keys stay in registers, 256 bins cut the range between the lowest and the
// highest key, and once the bin with the q-th largest holds no more than 64 keys, those are listed and one wave counts for
// each the ones in front of it (higher, or equal at a lower position).  A bin that is too full is cut into 256 again;
// keys that are all equal are taken in position order.  (Ranking up to 256 listed keys through LDS instead of one more
// pass took 16 us longer for 72 segments of 1457 normal scores.)  The picks are bits of a map of the segment, whose
// running count gives every pick its place in the ascending list.
template <int MODE, int BLOCK, int PER>
__global__ __launch_bounds__(BLOCK) void select_kernel(Dims d, int S, int budget, const float* g_all,
                                                       const int32_t* bounds_all,
                                                       const int32_t* quota_all, int32_t* idx_all,
                                                       uint32_t* flags_all, int n_words, GatherArgs ga) {
  constexpr bool FLAGS = MODE == SELECT_FLAGS, GATHER = MODE == SELECT_GATHER;
  constexpr int kW = BLOCK / 64, kCap = BLOCK * PER, kWords = kCap / 64, kPerLane = (kWords + 63) / 64;
  constexpr int kList = 64;  // keys that one wave ranks
  __shared__ __align__(16) BinsOrFar<BLOCK> bins;
  auto& hist = bins.hist;
  __shared__ uint2 list[kList];          // (key, position in the segment) of the keys in the bin
  __shared__ __align__(8) uint64_t picked[kWords], equal[kWords];
  __shared__ int before[kWords];         // picks in front of each word
  __shared__ int n_list;
  __shared__ uint2 red[kW];
  __shared__ int32_t rows[GATHER ? kGatherList : 1];
  const int unit = blockIdx.y, seg = GATHER ? (int)blockIdx.x / ga.parts : (int)blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t* bounds = bounds_all + (int64_t)unit * (S + 1);
  const int32_t* quota = quota_all + (int64_t)unit * S;
  const int a = bounds[seg], b = bounds[seg + 1], q = quota[seg];
  if (GATHER && ga.n_kept[unit] < 0) return;  // a scorer's bounded wait expired: nothing is kept
  // this workgroup's share of the segment's picks, by their place in ascending order
  int r0 = 0, r1 = q;
  if (GATHER && ga.parts > 1) {
    const int part = (int)blockIdx.x - seg * ga.parts;
    r0 = (int)((int64_t)q * part / ga.parts);
    r1 = (int)((int64_t)q * (part + 1) / ga.parts);
  }
  if (r0 >= r1) return;
  const int L = b - a;
  const float* g = g_all + (int64_t)unit * d.t_stride;
  uint32_t key[PER];
  const bool from_memory = L > kCap;
  if (q < L && !from_memory) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = i * BLOCK + (int)threadIdx.x;
      key[i] = e < L ? __float_as_uint(g[a + e]) : 0u;
    }
  }
  int out0 = 0;  // place of this segment's picks in the index list: the quotas before it
  if (!FLAGS) {
    for (int i = lane; i < seg; i += 64) out0 += quota[i];
    out0 = wave_sum(out0);
  }
  const Emit<FLAGS> emit{idx_all + (int64_t)unit * budget + out0,
                         FLAGS ? flags_all + (int64_t)unit * n_words : nullptr, r0, r1};
  if (q >= L) {  // whole segment kept
    for (int j = threadIdx.x; j < L; j += BLOCK) emit(j, a + j);
    if (GATHER) gather_rows<BLOCK>(d, ga, unit, out0, r0, r1, [&](int j) { return a + j; });
    return;
  }
  // a pick, the j-th of the segment
  auto take = [&](int j, int t) __attribute__((always_inline)) {
    emit(j, t);
    if (GATHER && j >= r0 && j < r1 && j - r0 < kGatherList) rows[j - r0] = t;
  };
  auto gather = [&]() __attribute__((always_inline)) {
    __syncthreads();
    gather_rows<BLOCK>(d, ga, unit, out0, r0, r1, [&](int j) __attribute__((always_inline)) {
      int t = rows[min(j - r0, kGatherList - 1)];
      asm volatile("" : "+v"(t));  // two loads, not one through a pointer to either memory
      if (j - r0 >= kGatherList) t = emit.out[j];
      return t;
    });
  };
  if (from_memory) {
    const bool vec = (d.t_stride & 3) == 0 && ((uintptr_t)g_all & 15) == 0;
    far_select<BLOCK>(bins.far, a, b, q, true,
                      [&](int t, uint32_t (&k)[4]) __attribute__((always_inline)) {
                        far_scores(g, a, b, t, vec, k);
                        return 0u;
                      },
                      take);
    if (GATHER) gather();
    return;
  }

  // range of the keys
  uint32_t lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = i * BLOCK + (int)threadIdx.x;
    key[i] = score_key(__uint_as_float(key[i]));
    if (e < L) {
      lo = min(lo, key[i]);
      hi = max(hi, key[i]);
    }
  }
  for (int i = threadIdx.x; i < 512; i += BLOCK) (&hist[0][0])[i] = 0;
  if (threadIdx.x == 0) n_list = 0;
  wave_min_max(lo, hi);
  if (lane == 0) red[wave] = make_uint2(lo, hi);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    lo = min(lo, red[w].x);
    hi = max(hi, red[w].y);
  }

  // keys in [lo, lo + 2^(sh + 8)) are cut into 256 bins of 2^sh; rem of them are still to be picked
  int sh = max(0, 24 - (int)__clz((int)((hi - lo) | 1u)));
  uint32_t span = hi - lo;  // highest offset that still belongs to the window
  int rem = q, n_bin = 0;
  for (int pass = 0;; ++pass) {
    int* h = hist[pass & 1];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t off = key[i] - lo;
      if (i * BLOCK + (int)threadIdx.x < L && key[i] >= lo && off <= span) atomicAdd(&h[off >> sh], 1);
    }
    __syncthreads();
    top_bin(h, lane, rem, lo, sh, n_bin);
    span = (1u << sh) - 1u;
    if (n_bin <= kList || n_bin == rem || sh == 0) break;
    sh = max(0, sh - 8);
    int* next = hist[(pass + 1) & 1];
    if (pass > 0) {  // the bins of two passes ago (every wave has read them: they were read before the last barrier)
      for (int i = threadIdx.x; i < 256; i += BLOCK) next[i] = 0;
      __syncthreads();
    }
  }
  // keys above lo + span are in, keys below lo are out, of the n_bin keys in between rem are to be picked
  const bool all = n_bin == rem, ranked = !all && n_bin <= kList;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (i * BLOCK >= L) break;
    const int e = i * BLOCK + (int)threadIdx.x;
    const bool valid = e < L && key[i] >= lo;
    const bool inside = valid && key[i] - lo <= span;
    const uint64_t top = __ballot(valid && (all || !inside)), mid = __ballot(inside);
    if (lane == 0) {
      picked[i * kW + wave] = top;
      if (!ranked) equal[i * kW + wave] = mid;
    }
    if (ranked && inside) list[atomicAdd(&n_list, 1)] = make_uint2(key[i], (uint32_t)e);
  }
  __syncthreads();
  const int words = (L + 63) / 64;
  if (ranked) {
    if (wave == 0) {
      const uint2 me = lane < n_bin ? list[lane] : make_uint2(0u, 0xFFFFFFFFu);
      int rank = 0;
      for (int j = 0; j < n_bin; ++j) {
        const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)me.x, j), e = (uint32_t)__builtin_amdgcn_readlane((int)me.y, j);
        rank += k > me.x || (k == me.x && e < me.y);
      }
      if (lane < n_bin && rank < rem) atomicOr((unsigned long long*)&picked[me.y >> 6], 1ull << (me.y & 63));
    }
    __syncthreads();
  } else if (!all) {  // equal keys: the first rem in position order
    if (wave == 0) {
      int c[kPerLane], t = 0;
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) {
        const int w = lane * kPerLane + i;
        c[i] = w < words ? __popcll(equal[w]) : 0;
        t += c[i];
      }
      int seen = wave_scan(t) - t;
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) {
        const int w = lane * kPerLane + i;
        if (w < words) {
          uint64_t m = equal[w];
          for (int drop = seen + c[i] - max(rem, seen); drop > 0; --drop) m &= ~(1ull << (63 - __clzll((long long)m)));
          picked[w] |= m;
        }
        seen += c[i];
      }
    }
    __syncthreads();
  }
  if (FLAGS) {  // the segment's map goes into the unit's, shifted to where the segment starts
    const uint32_t* map = (const uint32_t*)picked;
    const int s = a & 31;
    for (int w = threadIdx.x; w < 2 * words; w += BLOCK) {
      const uint32_t v = map[w];
      const int at = (a >> 5) + w;
      if (v << s) atomicOr(&emit.flags[at], v << s);
      if (s && v >> (32 - s)) atomicOr(&emit.flags[at + 1], v >> (32 - s));
    }
    return;
  }
  if (wave == 0) {
    int c[kPerLane], t = 0;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const int w = lane * kPerLane + i;
      c[i] = w < words ? __popcll(picked[w]) : 0;
      t += c[i];
    }
    int run = wave_scan(t) - t;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const int w = lane * kPerLane + i;
      if (w < words) before[w] = run;
      run += c[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (i * BLOCK >= L) break;
    const int w = i * kW + wave;
    if (w < words) {
      const uint64_t m = picked[w];
      if ((m >> lane) & 1ull) {
        const int j = before[w] + __popcll(m & ((1ull << lane) - 1ull)), t = a + i * BLOCK + (int)threadIdx.x;
        take(j, t);
      }
    }
  }
  if (GATHER) gather();
}

// Bits of word w (positions 32w .. 32w+31) that lie in [lo, hi).
__device__ __forceinline__ uint32_t range_bits(int w, int lo, int hi) {
  const int a = max(lo - w * 32, 0), b = min(hi - w * 32, 32);
  if (a >= b) return 0u;
  const uint32_t upto_b = b == 32 ? 0xFFFFFFFFu : (1u << b) - 1u;
  return upto_b & ~((1u << a) - 1u);
}

constexpr int kFinBlock = 1024;
constexpr int kFinWaves = kFinBlock / 64;
constexpr int kFinPer = 32;  // positions per thread whose keys stay in registers (T <= 32768)

__global__ __launch_bounds__(kFinBlock) void finalize_kernel(Dims d, const int32_t* seq_lens, int budget,
                                                             int n_sink, int n_last, const float* g_all,
                                                             uint32_t* flags_all, int n_words,
                                                             int32_t* idx_all) {
  __shared__ __align__(16) BinsOrFar<kFinBlock> bins;
  auto& hist = bins.hist;
  __shared__ int red[kFinWaves];
  __shared__ uint32_t red_lo[kFinWaves], red_hi[kFinWaves];
  __shared__ int wave_cnt[kFinWaves];
  __shared__ uint32_t bm[kFinBlock];  // the bitmap of a sequence of up to 32768 positions
  __shared__ uint2 list[64];          // (key, position) of the keys of the last bin
  __shared__ int n_list;
  const int unit = blockIdx.x;
  int l, b, h;
  unit_coords(d, unit, l, b, h);
  const int T = seq_len(d, seq_lens, b);
  const int kept = min(budget, T);
  const int sinks = min(n_sink, kept);
  const int last = min(n_last, kept - sinks);
  const float* g = g_all + (int64_t)unit * d.t_stride;
  uint32_t* flags = flags_all + (int64_t)unit * n_words;
  int32_t* idx = idx_all + (int64_t)unit * budget;
  const int nw = (T + 31) >> 5;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Up to 32768 positions the bitmap is worked on in LDS and the keys are read once into registers;
  // longer sequences keep the bitmap in memory and re-read the scores in every pass (far_select).
  const bool inreg = T <= kFinBlock * kFinPer;

  // union with the must-keep positions; size of the union
  int cnt = 0;
  if (inreg) bm[threadIdx.x] = 0u;
  for (int w = threadIdx.x; w < nw; w += kFinBlock) {
    const uint32_t f = flags[w] | range_bits(w, 0, sinks) | range_bits(w, T - last, T);
    if (inreg)
      bm[w] = f;
    else
      flags[w] = f;
    cnt += __popc(f);
  }
  cnt = wave_sum(cnt);
  if (lane == 0) red[wave] = cnt;
  __syncthreads();  // also orders the flag stores before the reads below
  cnt = 0;
#pragma unroll
  for (int w = 0; w < kFinWaves; ++w) cnt += red[w];
  const int deficit = kept - cnt;  // positions the duplicates left open; never negative
  const bool fill = deficit > 0;

  // Keys of the positions outside the set (0 = in the set or past the end; no score maps to 0).
  uint32_t kreg[kFinPer];
  auto key_at = [&](int t) __attribute__((always_inline)) -> uint32_t {
    if (t >= T) return 0u;
    return ((bm[t >> 5] >> (t & 31)) & 1u) ? 0u : score_key(g[t]);
  };
  if (fill && inreg) {
#pragma unroll
    for (int j = 0; j < kFinPer; ++j) kreg[j] = key_at(threadIdx.x + j * kFinBlock);
  }

  int rem = 0;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  if (inreg) {
    // The positions that fill the gap get their bits.  As in select_kernel: 256 bins over the range of the keys, the bin that
    // holds the deficit-th largest, a wave that ranks its keys, another 256 bins where they are too many.  93 -> 85 us per step
    // for 32 units of 6007 positions, 265 -> 246 for 504 ragged ones of up to 1617 (radix passes of 8 bits over a histogram per
    // wave before, three or four of them).
    if (fill) {
      uint32_t lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
      for (int j = 0; j < kFinPer; ++j) {
        if (j * kFinBlock < T && kreg[j]) {
          lo = min(lo, kreg[j]);
          hi = max(hi, kreg[j]);
        }
      }
      for (int i = threadIdx.x; i < 512; i += kFinBlock) (&hist[0][0])[i] = 0;
      if (threadIdx.x == 0) n_list = 0;
      wave_min_max(lo, hi);
      if (lane == 0) {
        red_lo[wave] = lo;
        red_hi[wave] = hi;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kFinWaves; ++w) {
        lo = min(lo, red_lo[w]);
        hi = max(hi, red_hi[w]);
      }
      int sh = max(0, 24 - (int)__clz((int)((hi - lo) | 1u)));
      uint32_t span = hi - lo;
      int n_bin = 0;
      rem = deficit;
      for (int pass = 0;; ++pass) {
        int* h = hist[pass & 1];
#pragma unroll
        for (int j = 0; j < kFinPer; ++j) {
          const uint32_t k = kreg[j];
          if (j * kFinBlock < T && k >= lo && k - lo <= span) atomicAdd(&h[(k - lo) >> sh], 1);  // (no key is 0, lo is at least 1)
        }
        __syncthreads();
        top_bin(h, lane, rem, lo, sh, n_bin);
        span = (1u << sh) - 1u;
        if (n_bin <= 64 || n_bin == rem || sh == 0) break;
        sh = max(0, sh - 8);
        int* next = hist[(pass + 1) & 1];
        if (pass > 0) {  // the bins of two passes ago
          for (int i = threadIdx.x; i < 256; i += kFinBlock) next[i] = 0;
          __syncthreads();
        }
      }
      // keys above lo + span fill the gap, and of the n_bin keys from lo to there rem
      const bool all = n_bin == rem, ranked = !all && n_bin <= 64;
#pragma unroll
      for (int j = 0; j < kFinPer; ++j) {
        const uint32_t k = kreg[j];
        const int t = threadIdx.x + j * kFinBlock;
        if (j * kFinBlock < T && k >= lo) {
          if (all || k - lo > span)
            atomicOr(&bm[t >> 5], 1u << (t & 31));
          else if (ranked)
            list[atomicAdd(&n_list, 1)] = make_uint2(k, (uint32_t)t);
        }
      }
      if (ranked) {
        __syncthreads();
        if (wave == 0) {
          const uint2 me = lane < n_bin ? list[lane] : make_uint2(0u, 0xFFFFFFFFu);
          int rank = 0;
          for (int q = 0; q < n_bin; ++q) {
            const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)me.x, q), e = (uint32_t)__builtin_amdgcn_readlane((int)me.y, q);
            rank += k > me.x || (k == me.x && e < me.y);
          }
          if (lane < n_bin && rank < rem) atomicOr(&bm[me.y >> 5], 1u << (me.y & 31));
        }
      } else if (!all) {  // the keys of the bin are equal: the first rem in index order
        int base_eq = 0;  // equal scores met so far (round j covers 1024 consecutive positions)
#pragma unroll
        for (int j = 0; j < kFinPer; ++j) {
          if (j * kFinBlock < T && base_eq < rem) {
            const int t = threadIdx.x + j * kFinBlock;
            const bool eq = kreg[j] == lo;
            const uint64_t be = __ballot(eq);
            if (lane == 0) red[wave] = __popcll(be);
            __syncthreads();
            int n_eq = base_eq + __popcll(be & below), tot = 0;
#pragma unroll
            for (int v = 0; v < kFinWaves; ++v) {
              if (v < wave) n_eq += red[v];
              tot += red[v];
            }
            if (eq && n_eq < rem) atomicOr(&bm[t >> 5], 1u << (t & 31));
            base_eq += tot;
            __syncthreads();
          }
        }
      }
      __syncthreads();
    }
    // ascending index list read off the bitmap: one word per thread
    const uint32_t f = bm[threadIdx.x];
    const int c = __popc(f);
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    if (lane == 63) wave_cnt[wave] = incl;
    __syncthreads();
    int slot = incl - c;
    for (int v = 0; v < wave; ++v) slot += wave_cnt[v];
    for (uint32_t m = f; m; m &= m - 1) idx[slot++] = threadIdx.x * 32 + __ffs((int)m) - 1;
    return;
  }

  // long sequences: the gap is filled and the list written in passes over the scores (26 units of 88025 positions: 85 us, 264
  // with radix passes and two barriers per 1024 positions; 10 of 131072: 116 and 388)
  const bool vec = (d.t_stride & 3) == 0 && ((uintptr_t)g_all & 15) == 0;
  far_select<kFinBlock>(bins.far, 0, T, deficit, fill,
                        [&](int t, uint32_t (&k)[4]) __attribute__((always_inline)) {
                          const uint32_t set = t < T ? flags[t >> 5] >> (t & 31) & 15u : 0u;
                          far_scores(g, 0, T, t, vec, k);
#pragma unroll
                          for (int i = 0; i < 4; ++i)
                            if ((set >> i) & 1u) k[i] = 0u;
                          return set;
                        },
                        [&](int slot, int t) __attribute__((always_inline)) { idx[slot] = t; });
}

}  // namespace

// The workgroups that select gather the rows as well: one launch less, and the latency of the selections that are still
// running hides behind the rows of the others.  us per step, with a gather kernel and without: 39.2 and 37.2 (8 fp32 units
// of 4096 positions, 1024 kept), 995 and 983 (256 units of 32768, 2048 kept), 167 and 162.5 (192 ragged units of up to 9001,
// 512 kept), 410 and 397 (1708 units of 1933, 144 kept), 141 and 136.5 (32 units of 27209, 3100 kept in 64 segments).  The gather
// kernel stays where the picks of a workgroup are many or few: long segments (8780 expected: 315 and 331 with short shares),
// most of the cache kept (256 units, 2048 of 2176: 171 and 177), a couple of rows per segment (93.5 and 94.8); and where
// the kept set is only known after finalize_kernel.
bool select_gathers(const ams_params* p) {
  const int S = p->n_segments, keep = p->budget < p->t_max ? p->budget : p->t_max;
  return p->n_sink == 0 && p->n_last == 0 && p->seg_delta == 0.f && (int64_t)p->t_max <= (int64_t)kGatherLongest * S &&
         (int64_t)keep * 2 < p->t_max && keep >= 8 * S;
}

hipError_t launch_select(const ams_params* p, const Dims& d, const int32_t* seq_lens, const float* g,
                         const int32_t* bounds, float* seg_mass, int32_t* quota, int32_t* idx,
                         int32_t* n_kept, uint32_t* flags, int n_words, hipStream_t s, bool quota_done,
                         const Gather* gather) {
  const int S = p->n_segments;
  if (S > kMaxSeg) return hipErrorInvalidValue;
  const bool must = p->n_sink > 0 || p->n_last > 0;
  if (must && (!flags || gather)) return hipErrorInvalidValue;
  if (!quota_done) {  // else the quotas, the tail of idx, the kept count and the cleared bitmap are already in place
    prof_mark("quota", s);
    hipLaunchKernelGGL(quota_kernel, dim3(d.units), dim3(64), 0, s, d, seq_lens, S, p->budget, p->q_min,
                       bounds, seg_mass, quota, idx, n_kept, p->n_sink, p->n_last,
                       must ? flags : nullptr, n_words);
  }
  prof_mark(gather ? "select_gather" : "select", s);
  // The expected segment length decides the shape of the selection workgroups (one wave: 1024 keys, 256 threads: 4096,
  // 512: 8192, 1024: 32768).  Segments differ by a factor of two or so, so a shape is left where longer ones would start
  // to miss the registers: 4096 expected takes 2272 us per step with 512 threads and 2328 with 1024 (2286 with 256, many
  // of whose segments go through memory); 2048 expected 998 with 256 and 1007 with 512; 512 expected 45.3 with 256 and
  // 46.7 with one wave; 136 expected 176.5 with one wave and 178.2 with 256.
  const double expect = p->seg_delta > 0.f
                            ? (p->l_max > 0 ? (double)p->l_max : (double)p->t_max * (double)p->seg_delta)
                            : (double)p->t_max / (double)S;
  GatherArgs ga{};
  if (gather) {
    ga = GatherArgs{gather->ks, gather->vs, gather->kd, gather->vd, gather->credit_src, gather->credit_dst, n_kept, p->budget, 1};
    // a small launch gives a segment's rows to several workgroups, which all select: 42.4 us per step for 8 fp32 units of 8
    // segments with one workgroup each, 37.2 with four (1024 rows of 512 bytes kept per unit); 59 and 52 for 6 units of 8
    // (at least 8 KB of keys to a share: what 256 threads move in two steps)
    const int rows = min(p->budget, d.t_max) / S;
    while ((int64_t)S * d.units * ga.parts < 512 && rows / (2 * ga.parts) * ga.ks.row_bytes >= 8192) ga.parts *= 2;
  }
  const dim3 grid(S * (gather ? ga.parts : 1), d.units);
#define AMS_SELECT(MODE, BLOCK, PER)                                                                               \
  hipLaunchKernelGGL((select_kernel<MODE, BLOCK, PER>), grid, dim3(BLOCK), 0, s, d, S, p->budget, g, bounds, quota, \
                     idx, flags, n_words, ga)
#define AMS_SELECT_SHAPE(MODE)             \
  if (expect <= 256.0)                     \
    AMS_SELECT(MODE, 64, 16);              \
  else if (expect <= 2560.0)               \
    AMS_SELECT(MODE, 256, 16);             \
  else if (expect <= 5120.0)               \
    AMS_SELECT(MODE, 512, 16);             \
  else                                     \
    AMS_SELECT(MODE, 1024, 32)
  if (must) {
    AMS_SELECT_SHAPE(SELECT_FLAGS);
    prof_mark("finalize", s);
    hipLaunchKernelGGL(finalize_kernel, dim3(d.units), dim3(kFinBlock), 0, s, d, seq_lens, p->budget, p->n_sink,
                       p->n_last, g, flags, n_words, idx);
  } else if (gather) {  // (select_gathers: no longer segments)
    if (expect <= 256.0)
      AMS_SELECT(SELECT_GATHER, 64, 16);
    else if (expect <= (double)kGatherLongest)
      AMS_SELECT(SELECT_GATHER, 256, 16);
    else
      return hipErrorInvalidValue;
  } else {
    AMS_SELECT_SHAPE(SELECT_LIST);
  }
#undef AMS_SELECT_SHAPE
#undef AMS_SELECT
  return hipGetLastError();
}

}  // namespace ams
