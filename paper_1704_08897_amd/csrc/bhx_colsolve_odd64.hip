// Column solve of 4095-node Dirichlet axes (64 rows a lane), which the FP32
// preconditioner alone takes: their odd extension has 8192 points, a power of
// two.  The form spills registers in a kernel that has the others as well
// (3000x3000 nodes, Neumann: 52 -> 56 us a pass).
//
// A source of its own, so that its code is an object of its own on the device:
// the other kernels' times depend on where they lie to about 1% (1231x877 258.0 ->
// 260.5 ms, 1100x600 116.0 -> 117.6 ms with two more kernels of any size, first or
// last, in their object; the same instructions, moved by 3 KB).
#include "bhx_colsolve.h"

namespace bhx {

hipError_t launch_colsolve_odd64(const Batch* B, int pass, int grid, int lds, hipStream_t st,
                                 hipEvent_t e1) {
  const hipEvent_t e0 = nullptr;
  if (pass == kPassZ)
    BHX_LAUNCH_T((k_colsolve<float, kPassZ, 3>), kColThreads, grid, lds, st, e0, e1, B, 0);
  else
    BHX_LAUNCH_T((k_colsolve<float, kPassC, 3>), kColThreads, grid, lds, st, e0, e1, B, 0);
  return hipGetLastError();
}

hipError_t set_colsolve_odd64_attributes() {
  const auto a = hipFuncAttributeMaxDynamicSharedMemorySize;
  const hipError_t e =
      hipFuncSetAttribute((const void*)k_colsolve<float, kPassC, 3>, a, kLdsDynMax);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_colsolve<float, kPassZ, 3>, a, kLdsDynMax);
}

}  // namespace bhx
