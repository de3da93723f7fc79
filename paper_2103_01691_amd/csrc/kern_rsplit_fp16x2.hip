// Resident-tile split product kernels, FP16X2.
#include "kern_rsplit.inl"

namespace mm {
hipError_t launch_rsplit_fp16x2(const ModePlan& p, const ModeArgs& a, const VortexW& w, hipStream_t s, hipEvent_t start,
                                hipEvent_t stop) {
  return rsplit_launch<KP_FP16X2>(p, a, w, s, start, stop);
}
}  // namespace mm
