// Usage u and base score g (Alg. 1 step 1; Sec. 3.2; Sec. 3.3 plug-in scorer).
//
// s[n][t] = q_n . k_t / sqrt(D) is a dense N x D by D x T contraction and runs on
// the matrix cores (32x32 MFMA tiles, token rows x query columns).  The row
// softmax needs every row's normaliser before a column can be finished, so the
// work is two sweeps over K:
//   sweep 1  per chunk of tokens, per query: running (max, sum of exp) in the
//            log2 domain, lane-local, merged per chunk          -> part_stats
//            (with the expected-attention scorers also the moment score -> g)
//   reduce   chunks merged in a fixed order                     -> (M_n, weights)
//   sweep 2  tiles recomputed, exp2(s - M_n) weighted by 1/(N Z_n) and summed
//            over the queries of each token                     -> u (and g)
// The score matrix itself never reaches memory.  The key-diversity and the
// value-weighted scorers add streaming kernels of their own at the end of the file.
#include "score_sweep.h"

namespace ams {
namespace {

// ---------------------------------------------------------------------------------------------
// Key-diversity score: g[t] = -cos(k_t, kbar), kbar the mean key of the unit.
// ---------------------------------------------------------------------------------------------
template <bool BF16>
__device__ __forceinline__ void widen8(const uint4& v, float (&x)[8], int& n) {
  if constexpr (BF16) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(w[i] << 16);
      x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
    n = 8;
  } else {
    x[0] = __uint_as_float(v.x);
    x[1] = __uint_as_float(v.y);
    x[2] = __uint_as_float(v.z);
    x[3] = __uint_as_float(v.w);
    n = 4;
  }
}

// partial key sums per chunk: ksum[unit][chunk][D] (double).  NORMALIZE: every key is divided by its
// length first (the redundancy-aware score needs the sum of the unit vectors; a zero key adds nothing).
template <bool BF16, int HD, bool NORMALIZE>
__global__ __launch_bounds__(kThreads) void keysum_kernel(ScoreArgs a, double* ksum) {
  constexpr int CPR = Tr<BF16, HD>::kRowBytes / 16, EPC = BF16 ? 8 : 4, RPI = kThreads / CPR;
  __shared__ double sm[kThreads][EPC];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int len = chunk_len(a, T), c0 = chunk * len;
  if (c0 >= T) return;
  const int col = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
  double s[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) s[e] = 0.0;
  // four rows per lane in flight (a row past the end re-reads the last one and is not added)
  constexpr int kRows = 4;
  const int t_end = min(T, c0 + len);
  for (int tb = c0 + r0; tb < t_end; tb += kRows * RPI) {
    uint4 v[kRows];
#pragma unroll
    for (int j = 0; j < kRows; ++j)
      v[j] = *(const uint4*)(kv_row(a.k, l, b, h, min(tb + j * RPI, T - 1)) + col * 16);
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      float x[8];
      int n;
      widen8<BF16>(v[j], x, n);
      double scale = 1.0;
      if (NORMALIZE) {  // the CPR lanes of a row are consecutive lanes of one wave
        float n2 = 0.f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) n2 = __builtin_fmaf(x[e], x[e], n2);
#pragma unroll
        for (int o = CPR / 2; o >= 1; o >>= 1) n2 += __shfl_xor(n2, o);
        scale = n2 > 0.f ? 1.0 / sqrt((double)n2) : 0.0;
      }
      if (tb + j * RPI < t_end) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) s[e] += (double)x[e] * scale;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < EPC; ++e) sm[threadIdx.x][e] = s[e];
  __syncthreads();
  if (threadIdx.x < CPR) {
    for (int e = 0; e < EPC; ++e) {
      double t = 0.0;
      for (int r = 0; r < RPI; ++r) t += sm[r * CPR + threadIdx.x][e];
      ksum[((int64_t)unit * a.n_chunks + chunk) * a.d.D + threadIdx.x * EPC + e] = t;
    }
  }
}

// MEAN_COS = false: g[t] = -cos(k_t, mean key).  MEAN_COS = true (ksum holds sums of unit vectors):
// g[t] = mean over s != t of cos(k_t, k_s) = (k_t / |k_t| . sum of unit vectors - 1) / (T - 1).
template <bool BF16, int HD, bool MEAN_COS>
__global__ __launch_bounds__(kThreads) void keydiff_kernel(ScoreArgs a, const double* ksum) {
  constexpr int CPR = Tr<BF16, HD>::kRowBytes / 16, EPC = BF16 ? 8 : 4, RPI = kThreads / CPR;
  __shared__ double kbar[128];
  __shared__ double kbar_norm;
  __shared__ float2 row_sums[kScoreChunk];  // per token: k . kbar and k . k
  const int unit = blockIdx.y, chunk = blockIdx.x;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int len = chunk_len(a, T), c0 = chunk * len;
  if (c0 >= T) return;
  const int nch = (T + len - 1) / len;
  if ((int)threadIdx.x < a.d.D) {
    double t = 0.0;
    for (int c = 0; c < nch; ++c) t += ksum[((int64_t)unit * a.n_chunks + c) * a.d.D + threadIdx.x];
    kbar[threadIdx.x] = MEAN_COS ? t : t / (double)T;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double n2 = 0.0;
    for (int d = 0; d < a.d.D; ++d) n2 += kbar[d] * kbar[d];
    kbar_norm = sqrt(n2);
  }
  __syncthreads();
  const int col = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
  float* g_row = a.g + (int64_t)unit * a.d.t_stride;
  float kb[EPC];  // this lane's channels of the mean key
#pragma unroll
  for (int e = 0; e < EPC; ++e) kb[e] = (float)kbar[col * EPC + e];
  // four rows per lane in flight: the loads are unconditional (a row past the end re-reads the last one)
  constexpr int kRows = 4;
  const int t_end = min(T, c0 + len);
  for (int tb = c0; tb < t_end; tb += kRows * RPI) {
    uint4 v[kRows];
#pragma unroll
    for (int j = 0; j < kRows; ++j)
      v[j] = *(const uint4*)(kv_row(a.k, l, b, h, min(tb + j * RPI + r0, T - 1)) + col * 16);
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      const int t = tb + j * RPI + r0;
      // a row's 128 products are summed in fp32 (8 per lane, then 16 or 32 lanes); the ratio is formed in double
      float dot = 0.f, nk = 0.f;
      float x[8];
      int n;
      widen8<BF16>(v[j], x, n);
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        dot = __builtin_fmaf(x[e], kb[e], dot);
        nk = __builtin_fmaf(x[e], x[e], nk);
      }
      // the CPR lanes of a row are consecutive lanes of one wave
#pragma unroll
      for (int o = CPR / 2; o >= 1; o >>= 1) {
        dot += __shfl_xor(dot, o);
        nk += __shfl_xor(nk, o);
      }
      if (col == 0 && t < t_end) row_sums[t - c0] = make_float2(dot, nk);
    }
  }
  __syncthreads();
  // one token per thread for the ratio, so that every lane works
  for (int t = c0 + threadIdx.x; t < min(T, c0 + len); t += kThreads) {
    const float2 r = row_sums[t - c0];
    if (MEAN_COS) {
      g_row[t] = (r.y > 0.f && T > 1) ? (float)(((double)r.x / sqrt((double)r.y) - 1.0) / (double)(T - 1)) : 0.f;
    } else {
      const double den = sqrt((double)r.y) * kbar_norm;
      g_row[t] = den > 0.0 ? (float)(-(double)r.x / den) : 0.f;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Value-weighted expected attention (Sec. 3.3 plug-in scorer): the log-moment scores e left in g by
// the second sweep become p = softmax over the cache, and g[t] = (p[t] + eps) * ||v_t||.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void esoftmax_part_kernel(ScoreArgs a, double2* part) {
  const int unit = blockIdx.y, chunk = blockIdx.x;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int len = chunk_len(a, T), c0 = chunk * len;
  if (c0 >= T) return;
  softmax_part(a.g + (int64_t)unit * a.d.t_stride + c0, min(len, T - c0), part + (int64_t)unit * a.n_chunks + chunk);
}

// Chunk statistics (maximum, sum of exp) of a unit's scores merged: every wave for itself, strided over the lanes, then a fixed
// tree.  (One thread in turn took 15 us for 73 chunks.)
__device__ __forceinline__ void merge_chunks(const ScoreArgs& a, const double2* part, int unit, int T, double& M, double& Z) {
  const int len = chunk_len(a, T), nch = (T + len - 1) / len, lane = threadIdx.x & 63;
  const double2* p = part + (int64_t)unit * a.n_chunks;
  M = -INFINITY;
  Z = 0.0;
  for (int c = lane; c < nch; c += 64) M = fmax(M, p[c].x);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) M = fmax(M, __shfl_xor(M, o));
  for (int c = lane; c < nch; c += 64) Z += p[c].y * exp(p[c].x - M);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) Z += __shfl_xor(Z, o);
}

// span: positions per workgroup, which need not be the sweeps' chunk.  Bound: the V stream.  A workgroup keeps one row per lane
// in flight, so it takes many of them: with the long chunks of a sweep that fills one round of workgroups 144 units of 16589
// positions took 185 us (3328 per workgroup) where spans of 1024 take 152.  Shorter chunks of such a sweep fit here as well.
template <bool BF16, int HD>
__global__ __launch_bounds__(kThreads) void vweight_kernel(ScoreArgs a, KvDev v, const double2* part, int span, float eps_f) {
  constexpr int CPR = Tr<BF16, HD>::kRowBytes / 16, EPC = BF16 ? 8 : 4, RPI = kThreads / CPR;
  __shared__ float norm2[kScoreChunk];  // per token: v . v
  const int unit = blockIdx.y;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int c0 = blockIdx.x * span;
  if (c0 >= T) return;
  double M, Z;
  merge_chunks(a, part, unit, T, M, Z);
  const double inv_z = 1.0 / Z, eps = (double)eps_f;
  const int col = threadIdx.x % CPR, r0 = threadIdx.x / CPR;
  float* g_row = a.g + (int64_t)unit * a.d.t_stride;
  for (int tb = c0; tb < min(T, c0 + span); tb += RPI) {
    const int t = tb + r0;
    float n2 = 0.f;  // 128 squares summed in fp32, the rest in double
    if (t < T) {
      const uint4 x4 = *(const uint4*)(kv_row(v, l, b, h, t) + col * 16);
      float x[8];
      int n;
      widen8<BF16>(x4, x, n);
#pragma unroll
      for (int e = 0; e < EPC; ++e) n2 = __builtin_fmaf(x[e], x[e], n2);
    }
    // the CPR lanes of a row are consecutive lanes of one wave
#pragma unroll
    for (int o = CPR / 2; o >= 1; o >>= 1) n2 += __shfl_xor(n2, o);
    if (col == 0 && t < T) norm2[t - c0] = n2;
  }
  __syncthreads();
  // one token per thread for the exponential, so that every lane works
  for (int t = c0 + threadIdx.x; t < min(T, c0 + span); t += kThreads)
    g_row[t] = (float)((exp((double)g_row[t] - M) * inv_z + eps) * sqrt((double)norm2[t - c0]));
}

template <bool BF16, int HD>
hipError_t launch_vweight(const ScoreArgs& a, const KvDev& v, char* ws, const WsLayout& wl, float eps, hipStream_t s) {
  const int span = min(a.chunk, a.k.layout == AMS_LAYOUT_DENSE ? wl.stream_chunk : wl.score_chunk_paged);
  hipLaunchKernelGGL((vweight_kernel<BF16, HD>), dim3(div_up(a.d.t_max, span), a.d.units), dim3(kThreads), 0, s, a, v,
                     (const double2*)(ws + wl.kbar), span, eps);
  return hipGetLastError();
}

template <bool BF16, int HD>
hipError_t launch_keydiff(const ScoreArgs& a, char* ws, const WsLayout& wl, hipStream_t s) {
  double* ksum = (double*)(ws + wl.kbar);
  const dim3 grid(a.n_chunks, a.d.units), blk(kThreads);
  prof_mark("keysum", s);
  hipLaunchKernelGGL((keysum_kernel<BF16, HD, false>), grid, blk, 0, s, a, ksum);
  prof_mark("keydiff", s);
  hipLaunchKernelGGL((keydiff_kernel<BF16, HD, false>), grid, blk, 0, s, a, (const double*)ksum);
  return hipGetLastError();
}

// Redundancy-aware score (Sec. 4 "Universality across diverse base scorers"): the mean cosine similarity of
// every key to the other keys of its unit (two streams of K: the sum of the unit vectors, then one dot product
// per key), its softmax over the cache, and g = lambda * (pooled) usage - (1 - lambda) * that softmax.
constexpr int kMixRun = 4 * kThreads;  // positions per workgroup of the kernel that mixes the two terms, four per thread
__global__ __launch_bounds__(kThreads) void redundancy_combine_kernel(ScoreArgs a, const double2* part, float mix_lambda,
                                                                       int pool_r) {
  __shared__ __align__(16) float tile[kMixRun + 2 * 31 + 4];
  const int unit = blockIdx.y;
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int c0 = blockIdx.x * kMixRun;
  if (c0 >= T) return;
  const float* u_row = a.u + (int64_t)unit * a.d.t_stride;
  float* g_row = a.g + (int64_t)unit * a.d.t_stride;
  const int first = c0 - pool_r, e = (int)threadIdx.x * 4;
  for (int i = threadIdx.x; i < kMixRun + 2 * pool_r; i += kThreads) {
    const int t = first + i;
    tile[i] = (t >= 0 && t < T) ? u_row[t] : 0.f;
  }
  float r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = c0 + e + i < T ? g_row[c0 + e + i] : 0.f;
  double M, Z;
  merge_chunks(a, part, unit, T, M, Z);
  const double inv_z = 1.0 / Z, lam = (double)mix_lambda, inv_full = 1.0 / (double)(2 * pool_r + 1);
  __syncthreads();
  // the mean of u over the positions t - r .. t + r that exist, stored as fp32: one walk for four positions
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
  for (int q = 0; q < 2 * pool_r + 4; q += 4) {
    const float4 x4 = *reinterpret_cast<const float4*>(&tile[e + q]);  // positions that do not exist hold zeros
    const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (q + j >= i && q + j <= i + 2 * pool_r) sum[i] += (double)x[j];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = c0 + e + i;
    if (t >= T) break;
    const int n = min(T - 1, t + pool_r) - max(0, t - pool_r) + 1;
    const float imp = (float)(n == 2 * pool_r + 1 ? sum[i] * inv_full : sum[i] / (double)n);
    g_row[t] = (float)(lam * (double)imp - (1.0 - lam) * (exp((double)r[i] - M) * inv_z));
  }
}

template <bool BF16, int HD>
hipError_t launch_redundancy(const ScoreArgs& a, char* ws, const WsLayout& wl, float mix_lambda, int kernel, bool cosines_done,
                             hipStream_t s) {
  double* ksum = (double*)(ws + wl.kbar);
  const dim3 grid(a.n_chunks, a.d.units), blk(kThreads);
  if (!cosines_done) {
    prof_mark("khat_sum", s);
    hipLaunchKernelGGL((keysum_kernel<BF16, HD, true>), grid, blk, 0, s, a, ksum);
    prof_mark("mean_cos", s);
    hipLaunchKernelGGL((keydiff_kernel<BF16, HD, true>), grid, blk, 0, s, a, (const double*)ksum);
  }
  const double2* soft = a.soft;
  if (!cosines_done) {
    prof_mark("esoftmax_part", s);  // the chunk statistics take the place of the key sums, which are used up
    hipLaunchKernelGGL(esoftmax_part_kernel, grid, blk, 0, s, a, (double2*)(ws + wl.kbar));
    soft = (const double2*)(ws + wl.kbar);
  }
  prof_mark("redundancy_combine", s);
  hipLaunchKernelGGL(redundancy_combine_kernel, dim3(div_up(a.d.t_max, kMixRun), a.d.units), blk, 0, s, a, soft, mix_lambda,
                     kernel > 1 ? kernel / 2 : 0);
  return hipGetLastError();
}

// Chunk statistics merged per query: the 1024 threads split into (query, contiguous range of
// chunks) pairs, the ranges are then combined in ascending order (fixed association) -> M_n and
// the per-query weights of the column sums.
// Latency bounds this kernel: a thread's range of up to two or up to eight chunks travels at once, a longer one four chunks at a
// time, and the credit before them.  us of the kernel with one chunk after the other and the credit last, with eight places at once
// in all ranges of up to eight, and as it is: 12.1, 12.8 and 12.2 (256 units of 32768, a chunk per thread), 11.0, 11.6 and 11.1 (the
// same with the expected attention), 5.6, 6.1 and 5.8 (causal window), 9.2, 7.6 and 7.6 (4 units of 10126, 80 chunks, five per
// thread), 11.5, 10.5 and 10.6 (10 of 87760), 23.5, 21.9 and 22.1 (112 of 131072, 224 queries).  A form for every power of two costs
// the causal one 0.2, the larger code being read in a kernel of 5 us; sixteen places at once lose (46.0 us per step, 42.9 with eight).
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void score_reduce_kernel(ScoreArgs a) {
  __shared__ float pm[kReduceThreads];
  __shared__ double pz[kReduceThreads];
  const int unit = blockIdx.x;
  if (unit == 0 && threadIdx.x == 0 && a.status) *a.status = 0;  // no bounded wait on this path
  int l, b, h;
  unit_coords(a.d, unit, l, b, h);
  const int T = seq_len(a.d, a.seq_lens, b);
  const int len = chunk_len(a, T), nch = (causal_t_end(a, T, a.causal) + len - 1) / len + (a.causal ? 1 : 0);
  double credit = 0.0;  // sum of the credit before the update (for the EMA normaliser), strided partials in a fixed tree
  if (a.csum) {         // first, so that the statistics travel meanwhile
    const float* c_row = a.credit + (int64_t)unit * a.d.t_stride;
    if ((a.d.t_stride & 3) == 0 && ((uintptr_t)a.credit & 15) == 0) {  // 16-byte loads, several in flight
      const float4* c4 = (const float4*)c_row;
      const int n4 = T >> 2;
#pragma unroll 8
      for (int q = threadIdx.x; q < n4; q += kReduceThreads) {
        const float4 v = c4[q];
        credit += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
      }
      for (int t = (n4 << 2) + threadIdx.x; t < T; t += kReduceThreads) credit += (double)c_row[t];
    } else {
      for (int t = threadIdx.x; t < T; t += kReduceThreads) credit += (double)c_row[t];
    }
  }
  const int parts = kReduceThreads / a.n_pad;
  const int n = threadIdx.x % a.n_pad, part = threadIdx.x / a.n_pad;
  if (part < parts) {
    const int per = (nch + parts - 1) / parts;
    const int c0 = part * per, c1 = min(nch, c0 + per);
    const float2* p = a.part + (int64_t)unit * (a.n_chunks + 1) * a.n_pad + n;
    float M = kNegInit;
    double Z = 0.0;
    auto all_at_once = [&](auto most) __attribute__((always_inline)) {
      constexpr int N = decltype(most)::value;
      float2 s[N];
#pragma unroll
      for (int i = 0; i < N; ++i) s[i] = c0 + i < c1 ? p[(int64_t)(c0 + i) * a.n_pad] : make_float2(kNegInit, 0.f);
#pragma unroll
      for (int i = 0; i < N; ++i) M = fmaxf(M, s[i].x);
#pragma unroll
      for (int i = 0; i < N; ++i) Z += (double)s[i].y * (double)__builtin_amdgcn_exp2f(s[i].x - M);
    };
    if (per <= 2) {
      all_at_once(std::integral_constant<int, 2>{});
    } else if (per <= 8) {
      all_at_once(std::integral_constant<int, 8>{});
    } else {
#pragma unroll 4
      for (int c = c0; c < c1; ++c) M = fmaxf(M, p[(int64_t)c * a.n_pad].x);
#pragma unroll 4
      for (int c = c0; c < c1; ++c) {
        const float2 s = p[(int64_t)c * a.n_pad];
        Z += (double)s.y * (double)__builtin_amdgcn_exp2f(s.x - M);
      }
    }
    pm[threadIdx.x] = M;
    pz[threadIdx.x] = Z;
  }
  __syncthreads();
  if ((int)threadIdx.x < a.n_pad) {
    float M = kNegInit;
    for (int q = 0; q < parts; ++q) M = fmaxf(M, pm[q * a.n_pad + n]);
    double Z = 0.0;
    for (int q = 0; q < parts; ++q) Z += pz[q * a.n_pad + n] * (double)__builtin_amdgcn_exp2f(pm[q * a.n_pad + n] - M);
    a.fin[(int64_t)unit * a.n_pad + n] = query_weights(a, n, T, M, Z, a.causal, true);
  }
  if (a.ksum && (int)threadIdx.x < a.d.D) {  // the unit's key sum takes the place of its first chunk's, for the second sweep
    double* k = a.ksum + (int64_t)unit * a.n_chunks * a.d.D + threadIdx.x;
    double t = 0.0;
#pragma unroll 8
    for (int c = 0; c < nch; ++c) t += k[(int64_t)c * a.d.D];
    *k = t;
  }
  if (a.csum) {
    __shared__ double cs[kReduceThreads / 64];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) credit += __shfl_xor(credit, o);
    if ((threadIdx.x & 63) == 0) cs[threadIdx.x >> 6] = credit;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < kReduceThreads / 64; ++w) t += cs[w];
      a.csum[unit] = t;
    }
  }
}

}  // namespace

hipError_t launch_score_reduce(const ScoreArgs& a, hipStream_t s) {
  prof_mark("score_reduce", s);
  hipLaunchKernelGGL(score_reduce_kernel, dim3(a.d.units), dim3(kReduceThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_first_sweep(const ScoreArgs& a, int nb, int head_dim, bool moments, bool bf16, hipStream_t s) {
  return first_sweep<false>(a, nb, head_dim, moments, bf16, s);
}

hipError_t launch_score(const ams_params* p, const Dims& d, const KvDev& k, const KvDev* v,
                        const int32_t* seq_lens,
                        const void* q, float* u, float* g, const float* credit, VcInfo* vc, char* ws,
                        const WsLayout& wl, hipStream_t s) {
  if (vc) vc->have = vc->cuts = false;
  ScoreArgs a;
  const bool causal = p->causal != 0 && d.W > 1;  // a window of one query sees everything anyway
  a.causal = causal;
  // the chunk sums of the second sweep would miss the tail blocks: the mass kernels form their own
  if (causal) vc = nullptr;
  a.vc_part = vc ? (double2*)(ws + wl.vc_part) : nullptr;
  a.credit = credit;
  a.csum = (vc && credit) ? (double*)(ws + wl.csum) : nullptr;
  a.ksum = nullptr;
  // softmax partials of a score that a sweep forms: the second sweep (mean cosines) leaves them where the sums of 64 positions
  // go later (it reads the statistics and the key sums itself), the first one (moment scores) takes the key sums' place,
  // which nobody uses then
  a.soft = nullptr;
  a.eps = p->mass_eps;
  a.k = k;
  a.d = d;
  a.seq_lens = seq_lens;
  a.q = (const char*)q;
  a.part = (float2*)(ws + wl.part_stats);
  a.fin = (float4*)(ws + wl.fin_stats);
  a.status = park_status_word(ws, wl);
  a.u = u;
  const bool paged = k.layout != AMS_LAYOUT_DENSE;
  a.n_chunks = paged ? wl.n_chunks_paged : wl.n_chunks;
  a.chunk = paged ? wl.score_chunk_paged : wl.score_chunk;
  // Chunks that fill one round of workgroups were cut from t_max, which may be a capacity: a shorter cache is shared by as many
  // workgroups.  us per step with chunks of a power of two, with the chunks as cut for t_max and with shares: 109, 158 and 90
  // (90 units of 5000 positions, t_max 20000), 102, 111 and 88 (32 of 13600 of 27209), 99, 109 and 87 (20 of 15000 of 30000, 224
  // queries); 48 pairs of shape and length take 0.46 to 1.0 of the power of two, 0.51 to 1.45 without the shares.
  a.even = !paged && wl.one_round;
  a.n_pad = wl.n_pad;
  // Batches whose sequences may differ in length: the workgroups count the chunks that exist (sweep_tile), where the launch has
  // more of them than run at once (162 and 143 us per step for 192 units of up to 9001; 12 shapes of 1536 to 2400 workgroups
  // take 0.84 to 1.0 of the time without).  The count costs 0.5 us per workgroup (93.5 and 95.2 for 48 x 3 units of up to 1376,
  // 52.3 and 53.3 for 2 x 3 of up to 20068).  From 1024 to 1536 workgroups it depends on how the lengths fall: 23 shapes take
  // 0.87 to 1.01, 0.99 on average, the stage calls of 64 units of up to 20011 (1280 workgroups) 208.3 us with it and 207.2
  // without, which is within the spread of their runs.  The line lies where none of the measured shapes loses.
  a.compact = d.B > 1 && d.B <= 64 && (int64_t)d.units * a.n_chunks >= 1536;
  // The second sweep merges the statistics itself where that is cheaper than a launch between the sweeps (1.2 us of gap and
  // 5 of its own): every workgroup reads its unit's partial statistics once more.  us per step, with the kernel and without:
  // 44.5 and 41.0 (8 fp32 units of 4096), 33.7 and 32.4 (9 units of 2105), 95.5 and 92 (24 fp32 units of 9804, 240
  // workgroups), 147.8 and 143.6 (32 units of 27209, 864 workgroups), 99.8 and 97.3 (48 units of 1376, 224 queries).  With up
  // to 2048 workgroups or 128 chunks there is no gain any more (828 units of 12608: 822 and 827), and with more than 32 KB of
  // partial statistics per unit every workgroup takes as long as the kernel (4 fp32 units of 7328, 112 queries: 61.6 and 63.9).
  // With the keys riding along every workgroup also adds up the chunks' key sums, 128 KB at 128 chunks of 128 channels; the same
  // line holds: 138 shapes (1 to 64 units of 4096 to 131072, 8 to 128 queries) take 0.92 to 1.01 of the time with the kernel.
  // Causal launches likewise, whose statistics have the tails' entry more (16 units of up to 2649: 88 and 82).
  a.fold = (int64_t)d.units * a.n_chunks <= 1024 && a.n_chunks * a.n_pad <= 4096;
  a.inv_sqrt_d = (float)(1.0 / sqrt((double)d.D));
  a.c2 = (float)(1.4426950408889634 / sqrt((double)d.D));
  const bool bf16 = p->kv_dtype == AMS_BF16;
  int mode = MODE_MEAN;
  a.g = nullptr;
  if (p->scorer == AMS_SCORER_MEAN_WINDOW) a.g = (g != u) ? g : nullptr;
  if (p->scorer == AMS_SCORER_LAST_QUERY) { mode = newest_share_lanes(d.W) ? MODE_LAST_LANES : MODE_LAST; a.g = g; }
  const bool vnorm = p->scorer == AMS_SCORER_EXPECTED_VNORM;
  if (vnorm && !v) return hipErrorInvalidValue;
  if (p->scorer == AMS_SCORER_EXPECTED || vnorm) { mode = MODE_EXPECTED; a.g = g; }
  if (vnorm && !causal) a.soft = (double2*)(ws + wl.kbar);
  const int nb = wl.n_pad / 32;
  bool oneread = false;
  int vc_stride = 0, vc_tokens = 0;
  bool vc_even = false;
  hipError_t e = hipSuccess;
  // AMS_SCORE_PATH_AUTO: the two sweeps, which are the faster of the two on every workload measured so far
  if (p->score_path == AMS_SCORE_PATH_ONE_READ)
    e = launch_score_oneread(p, d, k, seq_lens, q, u, g, credit, vc != nullptr, &vc_stride, &vc_tokens, ws, wl, s,
                             &oneread);
  if (e != hipSuccess) return e;
  if (!oneread && p->score_path == AMS_SCORE_PATH_ONE_READ) return hipErrorNotSupported;
  // the key-based scores ride along with the sweeps where these run plain over a bf16 cache
  const bool keys_ride = (p->scorer == AMS_SCORER_KEYDIFF || p->scorer == AMS_SCORER_REDUNDANCY) && bf16 && !causal;
  if (!oneread) {
    // Short caches with enough units to fill the chip: one workgroup per unit, one launch.  Not for the key-based scores, which
    // would have to stream K twice more (us per event with and without: 103 and 89 for 142 units of 1836 positions with the key
    // diversity, 164 and 114 for 128 of 4096, 358 and 249 for 300 of 3500 with the mean cosines).  And not for longer ones of
    // these caches where its single round leaves three CUs in eight or more idle and the sweeps run in one round too, two
    // workgroups to a CU or what fills it: there they take 0.75 to 1.0 of its time (seven lengths from 2817 to 4096 x 128 to 160
    // units x eight shapes of 8 to 128 queries, 64 and 128 channels, bf16 and fp32).  A second, nearly empty round costs them
    // more than they gain: up to 1.28 of its time (144 units of 3073, 152 of 3584, 176 of 2900).
    const bool thin = d.t_max > 2816 && d.units <= 160 && ((int64_t)d.units * a.n_chunks <= 512 || (!paged && wl.one_round));
    const bool want_unit = p->score_path == AMS_SCORE_PATH_ONE_LAUNCH ||
                           (p->score_path == AMS_SCORE_PATH_AUTO && d.units >= kUnitScorerMinUnits && !keys_ride && !thin);
    if (want_unit) {
      // The scorer's workgroups go on to the quotas (score_unit_kernel) where the 6 to 8 us at their end cost less than the launch.
      // Small bf16 tiles, of which a CU holds two that hide part of each other's end: up to three rounds; time without over time with
      // 1.02 to 1.06 for one, 1.04 to 1.09 for two (520 to 1024 units of 400 to 3500 positions), 1.00 to 1.07 for three (1040 to
      // 1536).  The others: one round, 1.03 to 1.08 (200 and 256 units of 400 to 3500, large bf16 tiles), 1.02 to 1.08 (130 and 256
      // fp32 units of 300 to 3000; four blocks of 128 channels 1.04 at 300 positions, 1.01 at 1000, 0.99 to 1.01 from 2000 on).  Two
      // rounds expose two such ends: 0.97 to 1.00 (264 to 512 units of 400 and 1500), fp32 0.98 to 0.99.  Past 2048 positions the
      // launch that they replace needs 512 threads a unit and costs more: there 1.00 to 1.01 (2176 and 3500), but for the tile that
      // fills the registers (128 channels, over 64 queries: 0.98 to 1.01).  Four rounds 0.98.
      const bool small = unit_tile_small(bf16, nb, d.D), two = bf16 && d.t_max > 2048 && (nb <= 2 || d.D == 64);
      const bool few = d.units <= (small ? 3 * 512 : two ? 2 * 256 : 256);
      const UnitCuts* cuts = vc && few ? vc->unit_cuts : nullptr;
      e = launch_score_unit(a, bf16, d.D, mode, cuts, s, &oneread);
      if (cuts && oneread) vc->cuts = true;
      if (e != hipSuccess) return e;
      vc_stride = 1;
      vc_tokens = kScoreChunk;
    }
    if (!oneread && p->score_path == AMS_SCORE_PATH_ONE_LAUNCH) return hipErrorNotSupported;
  }
  bool keys_done = false;
  if (!oneread && keys_ride) {
    a.g = g;
    a.ksum = (double*)(ws + wl.kbar);
    a.soft = (double2*)(ws + wl.sub);
    e = launch_key_sweeps(a, nb, d.D, p->scorer == AMS_SCORER_REDUNDANCY, s);
    a.ksum = nullptr;
    vc_stride = a.n_chunks;
    vc_tokens = a.chunk;
    vc_even = a.even;
    keys_done = true;
  } else if (!oneread) {
    const bool last = p->scorer == AMS_SCORER_LAST_QUERY, moments = mode == MODE_EXPECTED;
    e = causal ? launch_causal_first_sweep(a, nb, d.D, moments, bf16, s) : launch_first_sweep(a, nb, d.D, moments, bf16, s);
    if (e != hipSuccess) return e;
    ScoreArgs a2 = a;
    if (moments) a2.g = nullptr;  // the moment-based score has been written by the first sweep: the second one leaves g alone
    if (causal)
      e = last ? launch_causal_last_usage(a2, nb, d.D, mode, bf16, s) : launch_causal_usage(a2, nb, d.D, bf16, s);
    else
      e = last ? launch_last_usage(a2, nb, d.D, mode, bf16, s) : second_sweep<MODE_MEAN, false>(a2, nb, d.D, bf16, s);
    vc_stride = a.n_chunks;
    vc_tokens = a.chunk;
    vc_even = a.even;
  }
  if (e != hipSuccess) return e;
  if (vc) {
    vc->have = true;
    vc->stride = vc_stride;
    vc->tokens = vc_tokens;
    vc->even = vc_even;
  }
  if (vnorm) {
    if (!a.soft) {
      prof_mark("esoftmax_part", s);
      hipLaunchKernelGGL(esoftmax_part_kernel, dim3(a.n_chunks, d.units), dim3(kThreads), 0, s, a,
                         (double2*)(ws + wl.kbar));
    }
    prof_mark("vweight", s);
    if (d.D == 64)
      e = bf16 ? launch_vweight<true, 64>(a, *v, ws, wl, p->vnorm_eps, s) : launch_vweight<false, 64>(a, *v, ws, wl, p->vnorm_eps, s);
    else
      e = bf16 ? launch_vweight<true, 128>(a, *v, ws, wl, p->vnorm_eps, s) : launch_vweight<false, 128>(a, *v, ws, wl, p->vnorm_eps, s);
  }
  if (p->scorer == AMS_SCORER_REDUNDANCY) {
    a.g = g;
    if (d.D == 64)
      e = bf16 ? launch_redundancy<true, 64>(a, ws, wl, p->mix_lambda, p->score_kernel, keys_done, s)
               : launch_redundancy<false, 64>(a, ws, wl, p->mix_lambda, p->score_kernel, keys_done, s);
    else
      e = bf16 ? launch_redundancy<true, 128>(a, ws, wl, p->mix_lambda, p->score_kernel, keys_done, s)
               : launch_redundancy<false, 128>(a, ws, wl, p->mix_lambda, p->score_kernel, keys_done, s);
  }
  if (p->scorer == AMS_SCORER_KEYDIFF && !keys_done) {
    a.g = g;
    if (d.D == 64)
      e = bf16 ? launch_keydiff<true, 64>(a, ws, wl, s) : launch_keydiff<false, 64>(a, ws, wl, s);
    else
      e = bf16 ? launch_keydiff<true, 128>(a, ws, wl, s) : launch_keydiff<false, 128>(a, ws, wl, s);
  }
  return e;
}

}  // namespace ams
