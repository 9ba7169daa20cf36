// Eq. (1) + EMA credit (Sec. 3.2, 3.3; Alg. 1 steps 1-2) and the mass prefix sum with its cut
// points (Sec. 3.3 "Mass-based adaptive segmentation"; Alg. 1 step 3): thresholds k/S for exactly S
// segments, or k*Delta followed by the split / merge pass over the segment lengths.
//
// Positions are independent until the prefix sum, so the work is cut over the whole chip first and gathered per unit
// afterwards:
//
//   vc_sums_kernel       partial sums of max(u,0)+eps and of the old credit (only where the scorer
//                        has not left them: stage call, causal window, pooled usage); pools the usage on the way
//   mass_kernel          m = v/Z, c <- lambda c + (1-lambda) m, m_used, and the sum of m_used per 64 positions
//   sub_totals_kernel    those sums of a given m_used (stage call)
//   unit_cuts_kernel     one workgroup per unit: prefix over the sums of 64, the 64 positions that hold each cut, the
//                        split / merge pass, the segment masses and (fused step) the quotas
//
// ams_mass_segment_static runs the same kernels on the library's own scratch while the sums of 64 fit there; beyond that
// unit_cuts_kernel forms them itself, by the same additions in the same order.
//
// Normalisers: Z is the actual sum of max(u,0)+eps.  The credit normaliser sum(c_new) is taken as
// lambda * sum(c_old) + (1 - lambda) and the outer normaliser as 1: both identities hold exactly in
// real arithmetic (sum(m) = 1) and to ~1e-8 in floating point, far inside the fp32 tolerance, and
// they remove two dependent sweeps over T.
//
// Prefix: P(j) = C + p_local(j), C the prefix in front of the piece of 64 positions that holds j and p_local
// the scan inside it; the total of a piece IS p_local of its last position, so the "first position that reaches k/S"
// tests agree across pieces.  Everything that feeds a comparison is double.
#include <type_traits>

#include "ams_internal.h"
#include "mass_cuts.h"

namespace ams {
namespace {

// Partial sums of max(u,0)+eps and of the old credit per 1024 * ROUNDS positions, for the normalisers.
// Usage as Eq. (1) sees it: with pooling (App. A; Alg. 1 step 1 "optionally smooth") the mean of u over the positions
// t-r .. t+r that exist, rounded to fp32 like a stored intermediate and left in pooled_all for mass_kernel.  The chunk's
// scores and r more on either side are staged in LDS, from which a thread reads what its four positions see, 16 bytes at
// a time.
// Bound: the 8 (pooled: 12) bytes it moves per position.
template <int ROUNDS, bool POOL>
__global__ __launch_bounds__(kBlock) void vc_sums_kernel(MsArgs a, const float* u_all, const float* credit_all,
                                                          float eps_f, float* pooled_all) {
  constexpr int kRun = kBlock * 4 * ROUNDS;
  __shared__ double sm[kWaves];
  __shared__ __align__(16) float tile[POOL ? kRun + 2 * kMaxPoolR + 4 : 1];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int c0 = chunk * kRun;
  if (c0 >= T) return;
  const float* u = u_all + (int64_t)unit * a.d.t_stride;
  const float* credit = credit_all + (int64_t)unit * a.d.t_stride;
  double v = 0.0, c = 0.0;
  float cx[ROUNDS][4], ux[ROUNDS][4];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j0 = c0 + (r * kBlock + (int)threadIdx.x) * 4;
    load_run(credit, j0, T, a.vec, cx[r], 0.f);
    if (!POOL) load_run(u, j0, T, a.vec, ux[r], 0.f);
  }
  if (POOL) {
    const int r = a.pool_r, first = c0 - r;  // first = position of tile[0]
#pragma unroll 4
    for (int e = threadIdx.x; e < kRun + 2 * r; e += kBlock) {
      const int t = first + e;
      tile[e] = (t >= 0 && t < T) ? u[t] : 0.f;
    }
    __syncthreads();
    float* out = pooled_all + (int64_t)unit * a.d.t_stride;
#pragma unroll
    for (int rd = 0; rd < ROUNDS; ++rd) {
      const int e = (rd * kBlock + (int)threadIdx.x) * 4;
      float pooled[4];
      pool_run(tile, e, c0 + e, T, r, pooled);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (c0 + e + i < T) v += fmax((double)pooled[i], 0.0) + (double)eps_f;
      store_run(out, c0 + e, T, a.vec, pooled);
    }
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c += (double)cx[r][i];
      if (!POOL && c0 + (r * kBlock + (int)threadIdx.x) * 4 + i < T) v += fmax((double)ux[r][i], 0.0) + (double)eps_f;
    }
  v = block_sum(v, sm);
  c = block_sum(c, sm);
  if (threadIdx.x == 0) a.vc_part[(int64_t)unit * a.vc_stride + chunk] = make_double2(v, c);
}

// Eq. (1) and the EMA, position by position.  Bound: the 16 bytes per position it moves: 134 MB in 27 us (5.0 TB/s) for
// 256 units of 32768 positions, 235 MB in 46 us for 112 of 131072.  One workgroup per unit that also carried the prefix
// (scan, barrier and the next loads in turn) took 45 and 114 us, and 30 us for 8 units of 32768, where this takes 5 + 7
// with unit_cuts_kernel.  A workgroup takes ROUNDS runs of 1024 positions, all of their loads in flight before the normalisers are
// known; every wave adds up the unit's partial sums for itself, so no barrier stands between the loads and the stores.
template <int ROUNDS, bool TOTALS>
__global__ __launch_bounds__(kBlock) void mass_kernel(MsArgs a, const float* u_all, float* credit_all, float* m_used_all,
                                                      float lambda, float beta, float eps_f) {
  const int unit = blockIdx.y;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int first = blockIdx.x * ROUNDS * kBlock * 4;
  if (first >= T) return;
  const float* u = u_all + (int64_t)unit * a.d.t_stride;
  float* credit = credit_all + (int64_t)unit * a.d.t_stride;
  float* m_used = m_used_all + (int64_t)unit * a.d.t_stride;
  const int lane = threadIdx.x & 63;
  float ux[ROUNDS][4], cx[ROUNDS][4];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j0 = first + (r * kBlock + (int)threadIdx.x) * 4;
    load_run(u, j0, T, a.vec, ux[r], 0.f);
    load_run(credit, j0, T, a.vec, cx[r], 0.f);
  }
  const MassOf mass(a, unit, T, lambda, beta, eps_f);
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j0 = first + (r * kBlock + (int)threadIdx.x) * 4;
    float mu[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mu[i] = 0.f;
      if (j0 + i < T) mu[i] = mass(ux[r][i], cx[r][i]);
    }
    store_run(credit, j0, T, a.vec, cx[r]);
    store_run(m_used, j0, T, a.vec, mu);
    if (TOTALS) {
      double p[4];
      sub_scan(mu, p);
      if ((lane & (kSubLanes - 1)) == kSubLanes - 1 && j0 - (kSub - 4) < T)
        a.sub[(int64_t)unit * a.n_sub + j0 / kSub] = p[3];
    }
  }
}

// The sums of 64 positions of a given m_used, each with the largest prefix inside the piece.
__global__ __launch_bounds__(kBlock) void sub_totals_kernel(MsArgs a, const float* m_all) {
  const int unit = blockIdx.y;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int j0 = (blockIdx.x * kBlock + (int)threadIdx.x) * 4;
  if (blockIdx.x * kBlock * 4 >= T) return;
  float x[4];
  load_run(m_all + (int64_t)unit * a.d.t_stride, j0, T, a.vec, x, 0.f);
  double p[4];
  const double top = piece_scan(x, j0, T, p);
  if ((threadIdx.x & (kSubLanes - 1)) == kSubLanes - 1 && j0 - (kSub - 4) < T)
    ((double2*)a.sub)[(int64_t)unit * a.n_sub + j0 / kSub] = make_double2(p[3], top);
}

template <int BLOCK, int KIND, int ROUNDS = 2>
__global__ __launch_bounds__(BLOCK, BLOCK == 1024 ? 4 : 1) void unit_cuts_kernel(MsArgs a, const float* m_all, CutsOut o) {
  __shared__ CutsLds<BLOCK, KIND, ROUNDS> sm;
  float cx[ROUNDS][4];
  cuts_body<BLOCK, KIND, ROUNDS>(a, m_all, o, blockIdx.x, sm, sm.m, cx, 0.0, 0.0);
}

// 256 threads hold the prefix of 65536 positions and take 16 cuts a round, eight workgroups to a CU; longer caches and
// more cuts (in Delta mode all final segments are summed, 16 lanes to a segment) take 1024.
template <int KIND>
void launch_cuts(const MsArgs& a, const float* m_used, const CutsOut& o, hipStream_t s) {
  if (a.n_sub <= 1024 && (a.delta > 0.0 ? a.S : a.K) <= 33)
    hipLaunchKernelGGL((unit_cuts_kernel<256, KIND>), dim3(a.d.units), dim3(256), 0, s, a, m_used, o);
  else
    hipLaunchKernelGGL((unit_cuts_kernel<1024, KIND>), dim3(a.d.units), dim3(1024), 0, s, a, m_used, o);
}

// Runs of 1024 positions per workgroup of the position-wise kernels: four while that leaves two workgroups for every CU.
int mass_rounds(const Dims& d) { return (int64_t)d.units * div_up(d.t_max, 4096) >= 512 ? 4 : 1; }

template <bool TOTALS>
void launch_mass(const MsArgs& a, const ams_params* p, const float* u, float* credit, float* m_used, hipStream_t s) {
  prof_mark("mass_ema", s);
  if (mass_rounds(a.d) == 4)
    hipLaunchKernelGGL((mass_kernel<4, TOTALS>), dim3(div_up(a.d.t_max, 4096), a.d.units), dim3(kBlock), 0, s, a, u, credit,
                       m_used, p->ema_lambda, p->ema_beta, p->mass_eps);
  else
    hipLaunchKernelGGL((mass_kernel<1, TOTALS>), dim3(div_up(a.d.t_max, 1024), a.d.units), dim3(kBlock), 0, s, a, u, credit,
                       m_used, p->ema_lambda, p->ema_beta, p->mass_eps);
}

MsArgs make_args(const ams_params* p, const Dims& d, const int32_t* seq_lens, char* ws, const WsLayout& wl,
                 int32_t* bounds) {
  MsArgs a;
  a.d = d;
  a.seq_lens = seq_lens;
  a.S = p->n_segments;
  a.delta = (double)p->seg_delta;
  a.K = p->seg_delta > 0.f ? initial_segments(p->seg_delta) : p->n_segments;
  a.l_min = p->l_min;
  a.l_max = p->l_max;
  a.pool_r = p->pool_kernel > 1 ? p->pool_kernel / 2 : 0;
  a.vc_part = (double2*)(ws + wl.vc_part);
  a.vc_even = false;
  a.vc_stride = a.vc_tokens = 0;  // set by the launchers once it is known who leaves the sums
  a.sub = (double*)(ws + wl.sub);
  a.n_sub = div_up(p->t_max, kSub);
  a.bounds = bounds;
  a.vec = false;  // set by the launchers once the pointers are known
  return a;
}

// Scratch of ams_mass_segment_static: device memory that belongs to the library and lives as long as the
// process, one copy per GPU.  In host code the array's name is only a handle; the address that kernels and
// copies may use comes from hipGetSymbolAddress, once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

}  // namespace

hipError_t static_scratch(char** out) {
  constexpr int kMaxDevices = 64;
  static char* ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!ptr[dev]) {
    void* p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    ptr[dev] = (char*)p;
  }
  *out = ptr[dev];
  return hipSuccess;
}

// Partial sums for the normalisers, where the scorer has left none that fit; pooled usage goes to m_used.  Returns the
// usage that Eq. (1) sees and notes in a where the sums are.
static const float* own_sums(MsArgs& a, const ams_params* p, const float* u, const float* credit, float* m_used,
                             hipStream_t s) {
  const int rounds = mass_rounds(a.d);
  a.vc_tokens = kBlock * 4 * rounds;
  a.vc_stride = div_up(a.d.t_max, a.vc_tokens);
  const dim3 grid(a.vc_stride, a.d.units), blk(kBlock);
  prof_mark("vc_sums", s);
#define AMS_VC_SUMS(ROUNDS, POOL) \
  hipLaunchKernelGGL((vc_sums_kernel<ROUNDS, POOL>), grid, blk, 0, s, a, u, credit, p->mass_eps, m_used)
  if (a.pool_r > 0) {
    if (rounds == 4) AMS_VC_SUMS(4, true);
    else AMS_VC_SUMS(1, true);
    return m_used;
  }
  if (rounds == 4) AMS_VC_SUMS(4, false);
  else AMS_VC_SUMS(1, false);
#undef AMS_VC_SUMS
  return u;
}

hipError_t launch_ema(const ams_params* p, const Dims& d, const int32_t* seq_lens, const float* u,
                      float* credit, float* m_used, char* ws, const WsLayout& wl, hipStream_t s) {
  MsArgs a = make_args(p, d, seq_lens, ws, wl, nullptr);
  a.vec = d.t_stride % 4 == 0 && (((uintptr_t)u | (uintptr_t)credit | (uintptr_t)m_used) & 15) == 0;
  const float* usage = own_sums(a, p, u, credit, m_used, s);
  launch_mass<false>(a, p, usage, credit, m_used, s);
  return hipGetLastError();
}

hipError_t launch_segment(const ams_params* p, const Dims& d, const int32_t* seq_lens,
                          const float* m_used, int32_t* bounds, float* seg_mass, char* ws, const WsLayout& wl,
                          hipStream_t s) {
  MsArgs a = make_args(p, d, seq_lens, ws, wl, bounds);
  a.vec = d.t_stride % 4 == 0 && ((uintptr_t)m_used & 15) == 0;
  prof_mark("sub_totals", s);
  hipLaunchKernelGGL(sub_totals_kernel, dim3(div_up(d.t_max, kBlock * 4), d.units), dim3(kBlock), 0, s, a, m_used);
  CutsOut o{};
  o.seg_mass = seg_mass;
  prof_mark("unit_cuts", s);
  launch_cuts<CUTS_STAGE>(a, m_used, o, s);
  return hipGetLastError();
}

// ams_mass_segment_static.  The cuts do not depend on the workgroup's size (it only says how many pieces are held at once, and
// up to 1024 of them the first four waves of either size do the same), so the outputs are those of launch_segment bit for bit.
hipError_t launch_segment_static(const ams_params* p, const Dims& d, const int32_t* seq_lens,
                                 const float* m_used, int32_t* bounds, float* seg_mass, char* scratch, WsLayout wl,
                                 hipStream_t s) {
  wl.vc_part = wl.sub = 0;  // the sums of 64 are all that the scratch holds
  if ((int64_t)d.units * div_up(d.t_max, kSub) * (int64_t)sizeof(double2) <= (int64_t)kStaticScratchBytes)
    return launch_segment(p, d, seq_lens, m_used, bounds, seg_mass, scratch, wl, s);
  MsArgs a = make_args(p, d, seq_lens, scratch, wl, bounds);
  a.vec = d.t_stride % 4 == 0 && ((uintptr_t)m_used & 15) == 0;
  CutsOut o{};
  o.seg_mass = seg_mass;
  prof_mark("unit_cuts", s);
  // the reads of m_used bound this form: many units take the small workgroups, of which four fit a CU (1024 units of 8192
  // positions: 32 us per call with 1024 threads)
  if (a.n_sub <= 1024 && d.units >= 512)
    hipLaunchKernelGGL((unit_cuts_kernel<256, CUTS_OWN>), dim3(d.units), dim3(256), 0, s, a, m_used, o);
  else
    hipLaunchKernelGGL((unit_cuts_kernel<1024, CUTS_OWN>), dim3(d.units), dim3(1024), 0, s, a, m_used, o);
  return hipGetLastError();
}

// The arguments of the stages between the scores and the selection of a fused step.
hipError_t unit_cuts_args(const ams_params* p, const Dims& d, const int32_t* seq_lens, const float* u, float* credit, float* m_used,
                          int32_t* bounds, float* seg_mass, int32_t* quota, int32_t* idx, int32_t* n_kept, uint32_t* flags,
                          int n_words, char* ws, const WsLayout& wl, UnitCuts* out) {
  if (p->n_segments > kMaxSegments) return hipErrorInvalidValue;
  MsArgs& a = out->a;
  a = make_args(p, d, seq_lens, ws, wl, bounds);
  a.vec = d.t_stride % 4 == 0 && (((uintptr_t)u | (uintptr_t)credit | (uintptr_t)m_used) & 15) == 0;
  const bool must = p->n_sink > 0 || p->n_last > 0;
  if (must && !flags) return hipErrorInvalidValue;
  out->o = CutsOut{seg_mass, quota, idx, n_kept, must ? flags : nullptr, n_words, p->budget, p->q_min, p->n_sink,
                  p->n_last, (const int32_t*)park_status_word(ws, wl), u, credit, m_used, p->ema_lambda, p->ema_beta,
                  p->mass_eps};
  return hipSuccess;
}

// The one-launch scorer goes on to the quotas by itself where all of a unit's masses come from sums that it has: no pooling, few
// segments at thresholds k/S.
bool unit_scorer_cuts(const ams_params* p) {
  return p->pool_kernel <= 1 && p->seg_delta == 0.f && p->n_segments <= kStepMaxSeg;
}

// The fused step's mass / EMA / segmentation / quota stages, where the scorer has not done them.
hipError_t launch_unit_mass(const ams_params* p, const Dims& d, const int32_t* seq_lens, const UnitCuts& uc, const VcInfo& vc,
                            hipStream_t s) {
  if (vc.cuts) return hipSuccess;  // the scorer has done it
  MsArgs a = uc.a;
  CutsOut o = uc.o;
  const float* u = o.u;
  float *credit = o.credit, *m_used = o.m_used;
  const float* usage = u;
  // The scorer has left no sums (pooled usage, causal window): a workgroup per unit pools the usage of a short cache, forms its
  // normalisers and masses and finds the cuts, one launch where there were three.  us per step: 48.0 -> 42.2 (12 units of 1284,
  // the paper's options), 56.1 -> 50.7 (3 of 4093), 145 -> 137 (180 of 3731), 377 -> 362 (512 of 2000), 67.5 -> 64.8 (4 of 5105),
  // 376 -> 362 (256 of 8000), 718 -> 705 (512 of 8192).  From 4097 positions on 512 threads with 16 positions each; 1024 threads
  // with 8 spill (376 -> 372, 74 -> 77 for 32 units of 4791).  Same limits as CUTS_MASS below.
  const bool all = !(vc.have && a.pool_r == 0) && d.t_max <= 8192 && d.units <= 512;
  if (all) {  // (unit_cuts_kernel forms the sums)
  } else if (vc.have && a.pool_r == 0) {  // left by the scorer (sums of the unsmoothed usage)
    a.vc_stride = vc.stride;
    a.vc_tokens = vc.tokens;
    a.vc_even = vc.even;
  } else {
    usage = own_sums(a, p, u, credit, m_used, s);
  }
  o.u = usage;
  // Short caches: a workgroup holds all masses of its unit, eight positions per thread, and finds the cuts on chip; one launch
  // and one trip of the masses through memory less: 41.0 -> 39.2 us per step for 8 units of 4096, 32.4 -> 30.6 for 9 of 2105,
  // 172.2 -> 170.8 for 256 of 2176.  Up to 512 units; more of them keep the whole chip busy with the position-wise kernel
  // (1152 ragged units of 2435: 230.7 without and 235.3 with, 768 of 5384: 548 and 573).  At 16384 positions there is no gain
  // any more (24 units of 9804: 91 without and 97 with).
  if (all) {
    prof_mark("unit_mass_cuts", s);
    if (d.t_max <= 2048)
      hipLaunchKernelGGL((unit_cuts_kernel<256, CUTS_ALL>), dim3(d.units), dim3(256), 0, s, a, m_used, o);
    else if (d.t_max <= 4096)
      hipLaunchKernelGGL((unit_cuts_kernel<512, CUTS_ALL>), dim3(d.units), dim3(512), 0, s, a, m_used, o);
    else
      hipLaunchKernelGGL((unit_cuts_kernel<512, CUTS_ALL, 4>), dim3(d.units), dim3(512), 0, s, a, m_used, o);
    return hipGetLastError();
  }
  if (p->seg_delta == 0.f && p->n_segments <= kStepMaxSeg && d.t_max <= 8192 && d.units <= 512) {
    prof_mark("unit_mass_cuts", s);
    if (d.t_max <= 2048)
      hipLaunchKernelGGL((unit_cuts_kernel<256, CUTS_MASS>), dim3(d.units), dim3(256), 0, s, a, m_used, o);
    else if (d.t_max <= 4096)
      hipLaunchKernelGGL((unit_cuts_kernel<512, CUTS_MASS>), dim3(d.units), dim3(512), 0, s, a, m_used, o);
    else
      hipLaunchKernelGGL((unit_cuts_kernel<1024, CUTS_MASS>), dim3(d.units), dim3(1024), 0, s, a, m_used, o);
    return hipGetLastError();
  }
  launch_mass<true>(a, p, usage, credit, m_used, s);
  prof_mark("unit_cuts", s);
  if (p->seg_delta > 0.f || p->n_segments > kStepMaxSeg)
    launch_cuts<CUTS_GENERAL>(a, m_used, o, s);
  else
    launch_cuts<CUTS_STEP>(a, m_used, o, s);
  return hipGetLastError();
}

}  // namespace ams
