// Resident-tile product kernels, FP32.
#define MM_RES_C4 1
#include "kern_res.inl"

namespace mm {
hipError_t launch_res_f32(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  return res_launch<KP_F32>(p, a, s, start, stop);
}
hipError_t launch_res_batch_f32(const ResArgs* args, const ResItem* items, int count, size_t lds, hipStream_t s) {
  return res_batch_launch<KP_F32>(args, items, count, lds, s);
}
}  // namespace mm
