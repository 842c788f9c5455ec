// Device-wide building blocks: fills, exclusive scans into 64-bit offsets, folds.
#include "pm_scan.h"

using namespace pmscan;

namespace {

__global__ void k_iota(int64_t* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i;
}

// Grid folds in two launches: FOLD_G workgroups reduce strided slices of the partials
// to one pair each, then one workgroup reduces those.
constexpr int FOLD_T = 256;
constexpr int FOLD_G = 256;

__device__ inline void block_minmax(int& a, int& b) {
  __shared__ int smn[FOLD_T / 64], smx[FOLD_T / 64];
  for (int d = 32; d >= 1; d >>= 1) {
    a = min(a, __shfl_xor(a, d, 64));
    b = max(b, __shfl_xor(b, d, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    smn[threadIdx.x >> 6] = a;
    smx[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int q = 1; q < FOLD_T / 64; ++q) {
      a = min(a, smn[q]);
      b = max(b, smx[q]);
    }
}

__global__ __launch_bounds__(FOLD_T) void k_fold_max_part(const uint32_t* part, int64_t n,
                                                          uint32_t* out) {
  int a = 0, b = 0;  // values as non-negative float bit patterns fit int
  for (int64_t i = (int64_t)blockIdx.x * FOLD_T + threadIdx.x; i < n;
       i += (int64_t)FOLD_T * gridDim.x)
    b = max(b, (int)part[i]);
  block_minmax(a, b);
  if (threadIdx.x == 0) out[blockIdx.x] = (uint32_t)b;
}

}  // namespace

// max of non-negative float bit patterns (or any values below 2^31)
pm_status fold_max_u32(pm_context* c, const uint32_t* part, int64_t n, uint32_t* out) {
  const int g = (int)std::min<int64_t>(FOLD_G, std::max<int64_t>(1, (n + FOLD_T - 1) / FOLD_T));
  uint32_t* p2 = (uint32_t*)scratch(c, SC_FOLD, (size_t)2 * FOLD_G * sizeof(int32_t));
  if (!p2) return PM_ERR_NOMEM;
  hipLaunchKernelGGL(k_fold_max_part, dim3(g), dim3(FOLD_T), 0, c->stream, part, n, p2);
  hipLaunchKernelGGL(k_fold_max_part, dim3(1), dim3(FOLD_T), 0, c->stream, p2, (int64_t)g, out);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status run_iota(pm_context* c, int64_t* p, int64_t n) {
  if (n <= 0) return PM_OK;
  hipLaunchKernelGGL(k_iota, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, c->stream, p, n);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status launch_fill_u32(pm_context* c, uint32_t* p, int64_t n, uint32_t v) {
  if (n <= 0) return PM_OK;
  int64_t blocks = cdiv(n, 256);
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, c->stream, p,
                     n, v);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status launch_fill_u64(pm_context* c, uint64_t* p, int64_t n, uint64_t v) {
  if (n <= 0) return PM_OK;
  int64_t blocks = cdiv(n, 256);
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill<uint64_t>, dim3((unsigned)blocks), dim3(256), 0, c->stream, p,
                     n, v);
  PM_LAUNCH_CHECK();
  return PM_OK;
}

pm_status scan_u32(pm_context* c, const uint32_t* in, int64_t n, int64_t* out, int64_t* bsum) {
  return scan_generic(c, GetU32{in}, n, out, bsum);
}
