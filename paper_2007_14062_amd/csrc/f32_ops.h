// Pieces shared by the fp32 kernels: 64x64 tiles staged through registers into LDS, and the two ways
// the 32x32x2 fp32 matrix instruction reads them.  A work item has four waves; a wave owns a 32x32
// quarter of every block pair.
#ifndef BB_F32_OPS_H_
#define BB_F32_OPS_H_

#include "kernel_common.h"

namespace bb {

constexpr int kThreadsF32 = 256;
constexpr int kVecPerThreadF32 = kBlk * kDim / 4 / kThreadsF32;  // 4 x 16 bytes per thread and tile

// Global -> registers: one 64x64 fp32 tile, 16 bytes per lane per step, coalesced.
__device__ __forceinline__ void tile_fetch_f32(const float* tile, f32x4 (&regs)[kVecPerThreadF32]) {
#pragma unroll
  for (int i = 0; i < kVecPerThreadF32; ++i)
    regs[i] = *reinterpret_cast<const f32x4*>(tile + (i * kThreadsF32 + threadIdx.x) * 4);
}

// Registers -> LDS, rows padded so that the operand reads spread over the banks.
__device__ __forceinline__ void tile_store_f32(float* lds, const f32x4 (&regs)[kVecPerThreadF32]) {
#pragma unroll
  for (int i = 0; i < kVecPerThreadF32; ++i) {
    const int idx = i * kThreadsF32 + threadIdx.x;
    *reinterpret_cast<f32x4*>(lds + (idx >> 4) * kF32Stride + (idx & 15) * 4) = regs[i];
  }
}

// B operand of a product over d: this lane's row, contraction slot hf of step (u, e) is d = 8u + 4hf + e.
__device__ __forceinline__ void row_fragments_f32(const float* row, int hf, f32x4 (&f)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) f[u] = *reinterpret_cast<const f32x4*>(row + u * 8 + hf * 4);
}

// s = A B^T over d: A row `row_lds` per lane (row lane % 32 of a half tile), B as above.
__device__ __forceinline__ void mfma_rows_f32(const float* row_lds, int hf, const f32x4 (&b)[8], f32x16& s) {
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(row_lds + u * 8 + hf * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[u][e], s, 0, 0, 0);
  }
}

// acc[dt] += A^T B over the 32 rows of a half tile: A column dt*32 + col, and B an accumulator tile as it
// stands: slot hf of register r is row acc_row(r, hf), and A is read in that same order.
__device__ __forceinline__ void mfma_columns_f32(const float* half_tile, int hf, int col, const f32x16& b,
                                                 f32x16 (&acc)[2]) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
      const float a = half_tile[acc_row(r, hf) * kF32Stride + dt * 32 + col];
      acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b[r], acc[dt], 0, 0, 0);
    }
}

}  // namespace bb
#endif  // BB_F32_OPS_H_
