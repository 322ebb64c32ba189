// Device helpers and launch macros shared by the kernel sources.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <hsa/hsa.h>

#include "bhx_internal.h"

namespace bhx {

// 1 / x by the hardware reciprocal estimate refined with Newton-Raphson
// steps r <- r + r (1 - x r) (quadratic convergence from the estimate).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}
__device__ __forceinline__ float recip(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// Debug build (BHX_DEBUG_LDS_NAN=1): every transform kernel starts by
// filling its dynamic LDS with NaN, so a read of LDS that no thread of the
// block wrote shows up as NaN in the results instead of as stale values.  The
// dispatch packet gives the block's whole group segment; the dynamic part
// starts at smem.  A no-op in the normal build.
#ifndef BHX_DEBUG_LDS_NAN
#define BHX_DEBUG_LDS_NAN 0
#endif
__device__ __forceinline__ void debug_fill_lds(unsigned char* dyn) {
#if BHX_DEBUG_LDS_NAN
  const hsa_kernel_dispatch_packet_t* pkt =
      (const hsa_kernel_dispatch_packet_t*)__builtin_amdgcn_dispatch_ptr();
  const unsigned total = pkt->group_segment_size;
  const unsigned start =
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)dyn;
  double* d = (double*)dyn;
  for (unsigned i = threadIdx.x; start + 8 * (i + 1) <= total; i += blockDim.x)
    d[i] = __builtin_nan("");
  __syncthreads();
#else
  (void)dyn;
#endif
}

// Work item `it` of pass `p`: (instance << kItemShift) | local item.  A
// single-instance batch needs no table.
__device__ __forceinline__ int item_code(const Batch& B, int p, int it) {
  return B.count == 1 ? it : B.items[p][it];
}

// Persistent-grid item loop with an XCD-aware block order: consecutive
// logical blocks (neighbouring tiles / row groups) land on the same XCD,
// whose L2 then serves their shared halo rows.
__device__ __forceinline__ int logical_block() {
  const int nb = gridDim.x, b = blockIdx.x;
  if (nb % 8 != 0) return b;
  return (b & 7) * (nb >> 3) + (b >> 3);
}

}  // namespace bhx

// Launch on `st`; given events, through hipExtLaunchKernelGGL, whose dispatch
// records them at kernel start and end.
#define BHX_LAUNCH_T(kernel, threads, grid, lds, st, e0, e1, ...)                       \
  do {                                                                                \
    if ((e0) || (e1))                                                                 \
      hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, st, e0, e1, 0,    \
                            __VA_ARGS__);                                             \
    else                                                                              \
      hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, st, __VA_ARGS__);    \
  } while (0)
#define BHX_LAUNCH(kernel, grid, lds, st, e0, e1, ...) \
  BHX_LAUNCH_T(kernel, kThreads, grid, lds, st, e0, e1, __VA_ARGS__)
