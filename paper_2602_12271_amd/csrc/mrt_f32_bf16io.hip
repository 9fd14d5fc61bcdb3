// fp32 arithmetic and intermediates for bf16 storage.
#include "mrt_f32_kernels.hpp"

namespace mrt {

hipError_t run_f32_stage_r_bf16(const KParams& kp, dim3 grid, bool first, bool last, hipStream_t s) {
  return run_r_t<u16>(kp, grid, first, last, s);
}

hipError_t run_f32_stage_l_bf16(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  return run_l_t<u16>(kp, grid, last, s);
}

hipError_t run_f32_dense_bf16(const KParams& kp, dim3 grid, hipStream_t s) { return run_dense_t<u16>(kp, grid, s); }

}  // namespace mrt
