// fp32 path for fp32 storage, and the launchers of both storage types (bf16 storage: a file of its own,
// so that the two sets of kernels compile at the same time).
#include "mrt_f32_kernels.hpp"

namespace mrt {

hipError_t launch_f32_stage_r(const KParams& kp, int dtype, int nbh, bool first, bool last,
                              hipStream_t s) {
  dim3 grid(kp.ntk * kp.b1, kp.ntq, nbh);
  return dtype == MRT_F32 ? run_r_t<float>(kp, grid, first, last, s) : run_f32_stage_r_bf16(kp, grid, first, last, s);
}

hipError_t launch_f32_stage_l(const KParams& kp, int dtype, int nbh, bool last, hipStream_t s) {
  dim3 grid(kp.b2, kp.ntq, nbh);
  return dtype == MRT_F32 ? run_l_t<float>(kp, grid, last, s) : run_f32_stage_l_bf16(kp, grid, last, s);
}

hipError_t launch_f32_dense(const KParams& kp, int dtype, int nbh, hipStream_t s) {
  dim3 grid((kp.Nq + kDenseQ32 - 1) / kDenseQ32, nbh);
  return dtype == MRT_F32 ? run_dense_t<float>(kp, grid, s) : run_f32_dense_bf16(kp, grid, s);
}

}  // namespace mrt
