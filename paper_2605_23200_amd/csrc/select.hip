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
//                scores outside the set (the same selection over the unset positions; radix passes where the
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

// Segment longer than the registers hold: the scores are re-read from memory for every pass.
template <bool FLAGS, int BLOCK>
__device__ void select_from_memory(const float* g, int a, int b, int q, const Emit<FLAGS>& emit, int* hist,
                                   uint32_t* sel_prefix, int* sel_rem, int2* wave_cnt) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // radix select of the q-th largest key, 8 bits at a time from the top
  uint32_t prefix = 0, mask = 0;
  int rem = q;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int i = threadIdx.x; i < 256; i += BLOCK) hist[i] = 0;
    __syncthreads();
    for (int t = a + threadIdx.x; t < b; t += BLOCK) {
      const uint32_t k = score_key(g[t]);
      if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255], 1);
    }
    __syncthreads();
    if (wave == 0) {
      int hb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) hb[i] = hist[lane * 4 + i];
      const int s = hb[0] + hb[1] + hb[2] + hb[3];
      int incl = s;  // sum over lanes >= this one
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_down(incl, o);
        if (lane + o < 64) incl += v;
      }
      int cum = incl - s;  // keys in bins above this lane's
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        if (cum < rem && rem <= cum + hb[i]) {
          *sel_prefix = prefix | ((uint32_t)(lane * 4 + i) << shift);
          *sel_rem = rem - cum;
        }
        cum += hb[i];
      }
    }
    __syncthreads();
    prefix = *sel_prefix;
    rem = *sel_rem;
    mask |= 0xFFu << shift;
    __syncthreads();
  }
  // prefix = key of the q-th largest score; rem = how many of the keys equal to it are kept
  const uint32_t thr = prefix;
  int base_gt = 0, base_eq = 0;  // counts over the positions before the current tile
  for (int t0 = a; t0 < b; t0 += BLOCK) {
    const int t = t0 + threadIdx.x;
    uint32_t k = 0;
    const bool in = t < b;
    if (in) k = score_key(g[t]);
    const bool gt = in && k > thr, eq = in && k == thr;
    const uint64_t bgt = __ballot(gt), beq = __ballot(eq);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (lane == 0) wave_cnt[wave] = make_int2(__popcll(bgt), __popcll(beq));
    __syncthreads();
    int n_gt = base_gt + __popcll(bgt & below), n_eq = base_eq + __popcll(beq & below);
    int tot_gt = 0, tot_eq = 0;
#pragma unroll
    for (int w = 0; w < (BLOCK / 64); ++w) {
      const int2 c = wave_cnt[w];
      if (w < wave) {
        n_gt += c.x;
        n_eq += c.y;
      }
      tot_gt += c.x;
      tot_eq += c.y;
    }
    if (gt || (eq && n_eq < rem)) emit(n_gt + min(n_eq, rem), t);
    base_gt += tot_gt;
    base_eq += tot_eq;
    __syncthreads();
  }
}

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
  __shared__ __align__(16) int hist[2][256];
  __shared__ uint2 list[kList];          // (key, position in the segment) of the keys in the bin
  __shared__ __align__(8) uint64_t picked[kWords], equal[kWords];
  __shared__ int before[kWords];         // picks in front of each word
  __shared__ int n_list;
  __shared__ uint2 red[kW];
  __shared__ int2 wave_cnt[kW];
  __shared__ uint32_t mem_prefix;
  __shared__ int mem_rem;
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
  if (from_memory) {
    select_from_memory<FLAGS, BLOCK>(g, a, b, q, emit, &hist[0][0], &mem_prefix, &mem_rem, wave_cnt);
    if (GATHER) {
      __syncthreads();
      gather_rows<BLOCK>(d, ga, unit, out0, r0, r1, [&](int j) { return emit.out[j]; });
    }
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
        emit(j, t);
        if (GATHER && j >= r0 && j - r0 < kGatherList) rows[j - r0] = t;
      }
    }
  }
  if (GATHER) {
    __syncthreads();
    gather_rows<BLOCK>(d, ga, unit, out0, r0, r1,
                       [&](int j) { return j - r0 < kGatherList ? rows[j - r0] : emit.out[j]; });
  }
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
  __shared__ __align__(16) int hist[kFinWaves][256];
  __shared__ uint32_t sel_digit;
  __shared__ int sel_rem;
  __shared__ int red[kFinWaves];
  __shared__ uint32_t red_and[kFinWaves], red_or[kFinWaves];
  __shared__ int2 wave_cnt[kFinWaves];
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
  // longer sequences keep the bitmap in memory and re-read the scores in every pass.
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
    const uint32_t word = inreg ? bm[t >> 5] : flags[t >> 5];
    return ((word >> (t & 31)) & 1u) ? 0u : score_key(g[t]);
  };
  if (fill && inreg) {
#pragma unroll
    for (int j = 0; j < kFinPer; ++j) kreg[j] = key_at(threadIdx.x + j * kFinBlock);
  }

  // key of the deficit-th largest score among the positions outside the set
  uint32_t thr = 0xFFFFFFFFu;
  int rem = 0;
  if (fill && !inreg) {
    // bits that are the same in every key need no radix pass
    uint32_t k_and = 0xFFFFFFFFu, k_or = 0u;
    for (int t = threadIdx.x; t < T; t += kFinBlock) {
      const uint32_t k = key_at(t);
      if (k) {
        k_and &= k;
        k_or |= k;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      k_and &= __shfl_xor(k_and, o);
      k_or |= __shfl_xor(k_or, o);
    }
    if (lane == 0) {
      red_and[wave] = k_and;
      red_or[wave] = k_or;
    }
    __syncthreads();
    k_and = 0xFFFFFFFFu;
    k_or = 0u;
#pragma unroll
    for (int w = 0; w < kFinWaves; ++w) {
      k_and &= red_and[w];
      k_or |= red_or[w];
    }
    const uint32_t diff = k_and ^ k_or;
    thr = k_and;  // all keys equal: the threshold is that key
    rem = deficit;
    if (diff != 0) {
      const int hb = 31 - __clz(diff);  // highest bit in which two keys differ
      uint32_t mask = hb == 31 ? 0u : ~((2u << hb) - 1u);  // bits known so far
      uint32_t prefix = k_and & mask;
      int shift = max(hb - 7, 0);
      for (;;) {
        for (int i = threadIdx.x; i < kFinWaves * 256; i += kFinBlock) (&hist[0][0])[i] = 0;
        __syncthreads();
        for (int t = threadIdx.x; t < T; t += kFinBlock) {
          const uint32_t k = key_at(t);
          if (k && (k & mask) == prefix) atomicAdd(&hist[wave][(k >> shift) & 255], 1);
        }
        __syncthreads();
        if (wave == 0) {
          int hbin[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            hbin[i] = 0;
#pragma unroll
            for (int w = 0; w < kFinWaves; ++w) hbin[i] += hist[w][lane * 4 + i];
          }
          const int s = hbin[0] + hbin[1] + hbin[2] + hbin[3];
          int incl = s;  // sum over lanes >= this one
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_down(incl, o);
            if (lane + o < 64) incl += v;
          }
          int cum = incl - s;  // keys in bins above this lane's
#pragma unroll
          for (int i = 3; i >= 0; --i) {
            if (cum < rem && rem <= cum + hbin[i]) {
              sel_digit = (uint32_t)(lane * 4 + i);
              sel_rem = rem - cum;
            }
            cum += hbin[i];
          }
        }
        __syncthreads();
        // the digit may overlap bits that are already known; OR-ing it in is then a no-op for those bits
        prefix |= sel_digit << shift;
        rem = sel_rem;
        mask = shift == 0 ? 0xFFFFFFFFu : ~((1u << shift) - 1u);
        __syncthreads();
        if (shift == 0) break;
        shift = max(shift - 8, 0);
      }
      thr = prefix;
    }
  }

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
        red_and[wave] = lo;
        red_or[wave] = hi;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kFinWaves; ++w) {
        lo = min(lo, red_and[w]);
        hi = max(hi, red_or[w]);
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
    if (lane == 63) wave_cnt[wave].x = incl;
    __syncthreads();
    int slot = incl - c;
    for (int v = 0; v < wave; ++v) slot += wave_cnt[v].x;
    for (uint32_t m = f; m; m &= m - 1) idx[slot++] = threadIdx.x * 32 + __ffs((int)m) - 1;
    return;
  }

  // long sequences: one position per thread and round; a position is kept when its bit is set or its
  // score is above the threshold, and the first rem positions equal to the threshold join
  int base_keep = 0, base_eq = 0;
  for (int t0 = 0; t0 < T; t0 += kFinBlock) {
    const int t = t0 + threadIdx.x;
    bool keep = false, eq = false;
    if (t < T) {
      keep = (flags[t >> 5] >> (t & 31)) & 1u;
      if (fill && !keep) {
        const uint32_t k = score_key(g[t]);
        keep = k > thr;
        eq = k == thr;
      }
    }
    const uint64_t bk = __ballot(keep), be = __ballot(eq);
    if (lane == 0) wave_cnt[wave] = make_int2(__popcll(bk), __popcll(be));
    __syncthreads();
    int n_keep = base_keep + __popcll(bk & below), n_eq = base_eq + __popcll(be & below);
    int tot_keep = 0, tot_eq = 0;
#pragma unroll
    for (int v = 0; v < kFinWaves; ++v) {
      const int2 c = wave_cnt[v];
      if (v < wave) {
        n_keep += c.x;
        n_eq += c.y;
      }
      tot_keep += c.x;
      tot_eq += c.y;
    }
    if (keep)
      idx[n_keep + min(n_eq, rem)] = t;
    else if (eq && n_eq < rem)
      idx[n_keep + n_eq] = t;
    base_keep += tot_keep;
    base_eq += tot_eq;
    __syncthreads();
  }
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
