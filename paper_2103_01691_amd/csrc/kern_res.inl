// Kernel instances of the resident-tile products (resident.h) for one
// precision; included by kern_res_f64.hip and kern_res_f32.hip.  MM_RES_C4:
// the precision has the four-product form (FP32).
#include <hip/hip_ext.h>

#include <algorithm>

#include "resident.h"

namespace mm {
namespace {

__device__ __forceinline__ int64_t res_block() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// Register budgets: MF <= 2 runs four waves per SIMD (at most 128 registers),
// MF = 3, 4 two.  MF = 1 allows sixteen waves per workgroup (256 complex
// rows), the others eight.
template <int PR, int FORM, int MF, int NF, bool PH>
__global__ __launch_bounds__(MF == 1 ? 1024 : 512)
void res_kernel(ResArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  res_tile<PR, FORM, MF, NF, PH>(a, res_block(), lds);
}

template <int PR, int FORM, int KR>
__global__ __launch_bounds__(256) void res_run_kernel(ResArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  res_run_tile<PR, FORM, KR>(a, res_block(), lds);
}

template <int PR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PR == KP_F32 ? 4 : 3)))
void res_batch_kernel(const ResArgs* __restrict__ args,
                                                        const ResItem* __restrict__ items) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const ResItem it = items[blockIdx.x];
  const ResArgs& a = args[it.arg];
  switch (it.kind) {
#define MM_RK(F_, M_) \
  case F_ * 10 + M_: res_tile<PR, F_, M_, 1, false>(a, it.tile, lds); break;
    MM_RK(RF_C3, 1) MM_RK(RF_C3, 2) MM_RK(RF_C3, 3)
#if MM_RES_C4
    MM_RK(RF_C4, 1) MM_RK(RF_C4, 2) MM_RK(RF_C4, 3)
#endif
    MM_RK(RF_RC, 1) MM_RK(RF_RC, 2) MM_RK(RF_RC, 3)
    MM_RK(RF_RR, 1)
#undef MM_RK
#define MM_RK(M_) \
  case RES_KIND_NF2 + M_: res_tile<PR, RF_RR, M_, 2, false>(a, it.tile, lds); break;
    MM_RK(1) MM_RK(2) MM_RK(3)
#undef MM_RK
    default: break;
  }
}

typedef void (*ResFn)(ResArgs);

template <int PR, int FORM, int NF, bool PH>
ResFn res_fn(int mf) {
  switch (mf) {
    case 1: return &res_kernel<PR, FORM, 1, NF, PH>;
    case 2: return &res_kernel<PR, FORM, 2, NF, PH>;
    case 3: return &res_kernel<PR, FORM, 3, NF, PH>;
    case 4: return &res_kernel<PR, FORM, 4, NF, PH>;
    default: return nullptr;
  }
}

template <int PR, int FORM>
ResFn res_run_fn(int rows) {
  return rows == 32 ? &res_run_kernel<PR, FORM, 32> : &res_run_kernel<PR, FORM, 64>;
}

template <int PR>
ResFn res_pick(const ResPlan& p) {
  if (p.run) {
#if MM_RES_C4
    if (p.form == RF_C4) return res_run_fn<PR, RF_C4>(p.run);
#endif
    return p.form == RF_C3 ? res_run_fn<PR, RF_C3>(p.run)
                           : (p.form == RF_RC ? res_run_fn<PR, RF_RC>(p.run) : res_run_fn<PR, RF_RR>(p.run));
  }
  if (p.form == RF_C3) return p.ph ? res_fn<PR, RF_C3, 1, true>(p.mf) : res_fn<PR, RF_C3, 1, false>(p.mf);
#if MM_RES_C4
  if (p.form == RF_C4) return p.ph ? res_fn<PR, RF_C4, 1, true>(p.mf) : res_fn<PR, RF_C4, 1, false>(p.mf);
#endif
  if (p.form == RF_RC) return p.ph ? res_fn<PR, RF_RC, 1, true>(p.mf) : res_fn<PR, RF_RC, 1, false>(p.mf);
  return p.nf == 2 ? res_fn<PR, RF_RR, 2, false>(p.mf) : res_fn<PR, RF_RR, 1, false>(p.mf);
}

template <int PR>
hipError_t res_launch(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  ResFn fn = res_pick<PR>(p);
  if (!fn) return hipErrorInvalidDeviceFunction;
  if (p.lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid(p.grid_x, p.grid_y), block(p.threads);
  if (start || stop) hipExtLaunchKernelGGL(fn, grid, block, p.lds, s, start, stop, 0, a);
  else hipLaunchKernelGGL(fn, grid, block, p.lds, s, a);
  return hipGetLastError();
}

template <int PR>
hipError_t res_batch_launch(const ResArgs* args, const ResItem* items, int count, size_t lds, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)&res_batch_kernel<PR>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // (fewer than 2^32 threads per launch)
  for (int at = 0; at < count; at += 1 << 23) {
    hipLaunchKernelGGL(res_batch_kernel<PR>, dim3(std::min(count - at, 1 << 23)), dim3(256), lds, s, args, items + at);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace
}  // namespace mm
