// Kernel instances of the resident-tile split products (rsplit.h) for one
// precision; included by kern_rsplit_fp16x2.hip and kern_rsplit_bf16x3.hip.
#include <hip/hip_ext.h>

#include "rsplit.h"

namespace mm {
namespace {

// (BF16X3 on two N-fragments needs more than 128 registers: at most eight waves)
template <int PR, int FORM, int NF, bool PH>
__global__ __launch_bounds__(PR == KP_BF16X3 && NF == 2 ? 512 : 1024) void rsplit_kernel(ModeArgs a, VortexW w) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  rsplit_tile<PR, FORM, NF, PH>(a, w, blockIdx.x, (typename Tr<PR>::pc*)lds);
}

template <int PR>
hipError_t rsplit_launch(const ModePlan& p, const ModeArgs& a, const VortexW& w, hipStream_t s, hipEvent_t start,
                         hipEvent_t stop) {
  const bool ph = p.pro || p.epi;
  auto fn = p.rs == 2 ? (ph ? &rsplit_kernel<PR, RS_CC, 2, true> : &rsplit_kernel<PR, RS_CC, 2, false>)
                      : (ph ? &rsplit_kernel<PR, RS_CC, 1, true> : &rsplit_kernel<PR, RS_CC, 1, false>);
  if (p.rs_form == RS_RC) fn = &rsplit_kernel<PR, RS_RC, 2, false>;
  if (p.rs_form == RS_RR) fn = p.rs == 2 ? &rsplit_kernel<PR, RS_RR, 2, false> : &rsplit_kernel<PR, RS_RR, 1, false>;
  if (p.rs_lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.rs_lds);
    if (e != hipSuccess) return e;
  }
  if (start || stop) hipExtLaunchKernelGGL(fn, dim3(p.grid_x), dim3(p.threads), p.rs_lds, s, start, stop, 0, a, w);
  else hipLaunchKernelGGL(fn, dim3(p.grid_x), dim3(p.threads), p.rs_lds, s, a, w);
  return hipGetLastError();
}

}  // namespace
}  // namespace mm
