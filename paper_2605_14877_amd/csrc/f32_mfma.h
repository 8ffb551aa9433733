// Operand layouts shared by the fp32 matrix-core kernels (attention, calibration).
//
// v_mfma_f32_16x16x4_f32: D[16][16] += A[16][4] B[4][16].  Lane L = n + 16 g (n = L % 16, g = L / 16) supplies
// A[n][g] and B[g][n] and holds D[4 g + r][n] in register r = 0..3.
//
// Scores are formed transposed, S^T = K Q^T (A = 16 key rows, B = 16 query rows).  The order of the d products of a dot
// product is free as long as both operands agree, so MFMA step 4 j + i takes element 16 j + 4 g + i of the rows: a
// lane then loads its row in pieces of 16 bytes.  The operands go from memory straight into registers: the wavefronts
// of a workgroup walk different keys, so there is nothing for them to share in LDS.
#pragma once

#include "device_util.h"

namespace heatkv {
namespace f32m {

constexpr int TILE = 16;  // keys, or queries, of an MFMA tile

// 16 rows of D floats as an MFMA operand (A or B); rows past the `rows` valid ones repeat the last.
template <int D>
struct Rows {
  f32x4 v[D / 16];
  __device__ __forceinline__ void load(const float* base, int rows, int lane) {
    const float* p = base + min(lane & 15, rows - 1) * D + 4 * (lane >> 4);
#pragma unroll
    for (int j = 0; j < D / 16; ++j) v[j] = *reinterpret_cast<const f32x4*>(p + 16 * j);
  }
};

// S^T of 16 keys x 16 queries: register r of lane (n, g) is key 4 g + r, query n.
template <int D>
__device__ __forceinline__ f32x4 scores(const Rows<D>& k, const Rows<D>& q) {
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};  // two chains: half the depth of the sum
#pragma unroll
  for (int j = 0; j < D / 16; ++j) {
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(k.v[j][0], q.v[j][0], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(k.v[j][1], q.v[j][1], b, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(k.v[j][2], q.v[j][2], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(k.v[j][3], q.v[j][3], b, 0, 0, 0);
  }
  return a + b;
}

// Reductions over the four lane groups (lanes n, n + 16, n + 32, n + 48), in a fixed order.
__device__ __forceinline__ float max_groups(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float sum_groups(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

}  // namespace f32m
}  // namespace heatkv
