// Resident-tile split product kernels, BF16X3.
#include "kern_rsplit.inl"

namespace mm {
hipError_t launch_rsplit_bf16x3(const ModePlan& p, const ModeArgs& a, const VortexW& w, hipStream_t s, hipEvent_t start,
                                hipEvent_t stop) {
  return rsplit_launch<KP_BF16X3>(p, a, w, s, start, stop);
}
}  // namespace mm
