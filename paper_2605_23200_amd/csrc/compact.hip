// Gather-compact of the kept rows (Alg. 1 step 6: K' = K[idx], V' = V[idx]); with a paged
// destination this is the head-wise compaction copy of App. E.  Pure byte movement: a row of
// head_dim elements is moved by row_bytes/16 consecutive lanes with 16-byte accesses, so every
// row is one fully used 256- or 512-byte burst on both sides.
#include "ams_internal.h"

namespace ams {
namespace {

constexpr int kBlock = 256;

template <int kRowsPerBlock>
__global__ __launch_bounds__(kBlock) void compact_kernel(Dims d, KvDev ks, KvDev vs, KvDev kd, KvDev vd,
                                                         int budget, const int32_t* idx_all,
                                                         const int32_t* n_kept_all,
                                                         const float* credit_src, float* credit_dst) {
  const int unit = blockIdx.y;
  int l, b, h;
  unit_coords(d, unit, l, b, h);
  // a count above the budget or an index outside the cache (a caller's mistake when the stage is
  // used on its own) must not turn into an access outside the buffers: the count is clamped and
  // such a row is skipped
  const int n = min(n_kept_all[unit], min(budget, d.t_max));
  const int j0 = blockIdx.x * kRowsPerBlock;
  if (j0 >= n) return;
  const int32_t* idx = idx_all + (int64_t)unit * budget;
  const int lanes_per_row = ks.row_bytes / 16;
  const int rows_per_pass = kBlock / lanes_per_row;
  const int sub = threadIdx.x % lanes_per_row, r = threadIdx.x / lanes_per_row;
  for (int jj = r; jj < kRowsPerBlock; jj += rows_per_pass) {
    const int j = j0 + jj;
    if (j >= n) break;
    const int t = idx[j];
    if (t < 0 || t >= d.t_max) continue;
    const uint4 kx = *(const uint4*)(kv_row(ks, l, b, h, t) + sub * 16);
    const uint4 vx = *(const uint4*)(kv_row(vs, l, b, h, t) + sub * 16);
    *(uint4*)(kv_row(kd, l, b, h, j) + sub * 16) = kx;
    *(uint4*)(kv_row(vd, l, b, h, j) + sub * 16) = vx;
  }
  if (credit_src && credit_dst && threadIdx.x < kRowsPerBlock) {
    const int j = j0 + threadIdx.x;
    if (j < n && idx[j] >= 0 && idx[j] < d.t_max)
      credit_dst[(int64_t)unit * budget + j] = credit_src[(int64_t)unit * d.t_stride + idx[j]];
  }
}

}  // namespace

hipError_t launch_compact(const ams_params* p, const Dims& d, const KvDev& ks, const KvDev& vs,
                          const KvDev& kd, const KvDev& vd, const int32_t* idx, const int32_t* n_kept,
                          const float* credit_src, float* credit_dst, hipStream_t s) {
  const int max_keep = p->budget < d.t_max ? p->budget : d.t_max;
  prof_mark("compact", s);
  const bool paged = ks.layout == AMS_LAYOUT_PAGED || kd.layout == AMS_LAYOUT_PAGED;
#define AMS_COMPACT(ROWS)                                                                                        \
  hipLaunchKernelGGL((compact_kernel<ROWS>), dim3((max_keep + ROWS - 1) / ROWS, d.units), dim3(kBlock), 0, s, d, \
                     ks, vs, kd, vd, p->budget, idx, n_kept, credit_src, credit_dst)
  // One pass of the workgroup over its rows (two for rows of 512 bytes) where the launch is small or most of the cache is
  // kept, so that no pass waits for the indices of the one before: 45.4 -> 42.4 us per step for 8 fp32 units of 1024 kept
  // rows, 70.4 -> 68.8 for 8 bf16 units of 2048, 177.4 -> 172.8 for 256 units that keep 2048 of 2176.  A large gather of
  // few rows (256 units, 2048 of 32768: 1008 against 1011) and paged caches (5994 against 5997) do not gain and keep 64.
  // (All index and row reads of 64 rows ahead of their stores is slower: 177 -> 225, the stores come in bursts.)
  const bool small = (int64_t)d.units * max_keep < 65536, most = (int64_t)max_keep * 2 >= d.t_max;
  if (paged || !(small || most))
    AMS_COMPACT(64);
  else if (ks.row_bytes < 256)
    AMS_COMPACT(32);
  else
    AMS_COMPACT(16);
#undef AMS_COMPACT
  return hipGetLastError();
}

}  // namespace ams
