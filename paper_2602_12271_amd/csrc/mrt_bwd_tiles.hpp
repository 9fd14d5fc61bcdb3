// Building blocks shared by the bf16 kernels of the backward pass (mrt_bwd_bf16.hip, mrt_bwd_waves_bf16.hip).
#pragma once
#include "mrt_bf16_tiles.hpp"

namespace mrt {
namespace {

// Matrix operand from a row-major LDS tile X[j][i]: lane (g, c) receives column i0 + c of the rows
// j = 16 (e / 4) + 4 g + e % 4, e = 0 .. 7 (the slots of pv_step).
template <int PITCH>
__device__ inline bf16x8 ld_columns(const u16* tile, int i0, int lane) {
  const int g = lane >> 4, s = lane & 15;
  const u16* at = tile + (4 * g + (s >> 2)) * PITCH + i0 + 4 * (s & 3);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(ld_lds_tr(at), ld_lds_tr(at + 16 * PITCH), 0, 1, 2, 3, 4, 5, 6, 7));
}

// A lane's D/16 accumulator tiles as fp32: 8 consecutive features at 32q + 8g per pair of tiles.
// The same rows with non-temporal stores: gradients that no later kernel of the call reads or adds
// to (they would only displace the workspace arrays from the caches).
template <int D>
__device__ inline void store_rows_f32_nt(float* row, const f32x4* acc, float mul, int g) {
#pragma unroll
  for (int q = 0; q < D / 32; ++q) {
    f32x4* p = (f32x4*)(row + 32 * q + 8 * g);
    __builtin_nontemporal_store(acc[2 * q] * mul, p);
    __builtin_nontemporal_store(acc[2 * q + 1] * mul, p + 1);
  }
}
template <int D>
__device__ inline void store_rows_f32(float* row, const f32x4* acc, float mul, int g, bool add) {
#pragma unroll
  for (int q = 0; q < D / 32; ++q) {
    f32x4* p = (f32x4*)(row + 32 * q + 8 * g);
    f32x4 a = acc[2 * q] * mul, b = acc[2 * q + 1] * mul;
    if (add) { a += p[0]; b += p[1]; }
    p[0] = a;
    p[1] = b;
  }
}

// A lane's row of D/16 accumulator tiles into a workspace array of either type (overwriting).
template <int D>
__device__ inline void store_ws_row(float* row, const f32x4* acc, float mul, int g) {
  store_rows_f32<D>(row, acc, mul, g, false);
}
template <int D>
__device__ inline void store_ws_row(u16* row, const f32x4* acc, float mul, int g) {
  store_rows<D>(row, acc, mul, g);
}

// Workgroups of `kernel` the current device keeps resident at once (its compute units times the
// workgroups of `threads` threads that fit one): the size of a persistent grid.
template <typename K>
inline int resident_workgroups(K kernel, int threads) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  return per_cu * cus;
}

}  // namespace
}  // namespace mrt
