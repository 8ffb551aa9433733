// Operand layouts of the kernels on the fp32 matrix instructions (attention, calibration), and the softmax arithmetic that
// those on three bf16 parts (f32_split.h) share with them.
//
// v_mfma_f32_16x16x4_f32: D[16][16] += A[16][4] B[4][16].  Lane L = n + 16 g (n = L % 16, g = L / 16) supplies
// A[n][g] and B[g][n] and holds D[4 g + r][n] in register r = 0..3.
//
// Scores are formed transposed, S^T = K Q^T (A = 16 key rows, B = 16 query rows).  The order of the d products of a dot
// product is free as long as both operands agree, so MFMA step 4 j + i takes element 16 j + 4 g + i of the rows: a
// lane then takes its row in pieces of 16 bytes.
//
// Two things about this chip shape the kernels.  (1) fp32 matrix instructions do not overlap with vector-ALU
// instructions, not even those of another wavefront (loops of 32 MFMAs 1.85 ms, of 128 FMAs 0.63 ms, of both 2.84 ms; with
// bf16 MFMAs 1.75, 0.57 and 1.90; profiles/f32_kernel_traces_and_overlap.txt): every vector instruction of a tile step adds to its 1024 (scores, d = 128) or 2048
// cycles, hence the care with addresses below.  (2) The vector L1 coalesces neighbouring lanes only, and in the operand
// layout those are in different rows: a fetch of keys straight into it costs 64 accesses per instruction, 2048 cycles
// of the L1 for the tiles of four wavefronts, twice their score MFMAs.  So a wavefront fetches its key tiles into an LDS
// stage of its own with whole rows side by side, and takes the operand from there.
#pragma once

#include "device_util.h"
#include "tile_lds.h"

namespace heatkv {
namespace f32m {

constexpr int TILE = 16;  // keys, or queries, of an MFMA tile

// A load is written as scalar base + 32-bit lane offset + immediate.  The base is hidden from the optimiser, which
// otherwise folds the two into 64-bit vector arithmetic of its own for every load.
typedef const __attribute__((address_space(1))) char* GlobalBytes;
__device__ __forceinline__ GlobalBytes scalar_base(const float* p) {
  GlobalBytes b = (GlobalBytes)p;
  asm volatile("; scalar base" : "+s"(b));
  return b;
}
__device__ __forceinline__ f32x4 load16(GlobalBytes base, unsigned off) {
  return *(const __attribute__((address_space(1))) f32x4*)(base + off);
}

// 16 rows of D floats as an MFMA operand (A or B); rows past the `rows` valid ones repeat the last.
template <int D>
struct Rows {
  f32x4 v[D / 16];
  __device__ __forceinline__ void load(const float* p, int rows, int lane) {
    const GlobalBytes base = scalar_base(p);
    const unsigned off = (min(lane & 15, rows - 1) * D + 4 * (lane >> 4)) * 4;
#pragma unroll
    for (int j = 0; j < D / 16; ++j) v[j] = load16(base, off + 64 * j);
  }
};

// A wavefront's LDS stage for one tile of 16 key rows.  Copies of 1 KB (tile_lds.h: copy_1k; the compiler does not see
// them as LDS stores or count them); the 16-byte chunks of a row are XORed with the row number, so that the 16 lanes
// that read the same chunk of 16 rows (rows start on the same bank) cover all 64 banks.
template <int D>
struct KeyStage {
  static constexpr int BYTES = TILE * D * 4;
  static constexpr int COPIES = BYTES / 1024;
  static constexpr int CPR = D / 4;  // chunks per row
  unsigned lds;                      // LDS byte address of the stage
  int off[COPIES];                   // lane offsets of the copies of a full tile
  __device__ __forceinline__ KeyStage(const char* stage, int lane) {
    lds = __builtin_amdgcn_readfirstlane(
        static_cast<unsigned>(reinterpret_cast<unsigned long long>((__attribute__((address_space(3))) const char*)stage)));
#pragma unroll
    for (int j = 0; j < COPIES; ++j) off[j] = offset(j, lane, TILE);
  }
  static __device__ __forceinline__ int offset(int j, int lane, int rows) {
    const int row = (64 * j + lane) / CPR;
    return min(row, rows - 1) * (4 * D) + (((lane & (CPR - 1)) ^ row) << 4);
  }
  // Starts the copy of rows base[0 .. rows); the stage must have been taken.
  __device__ __forceinline__ void fill(const float* base, int rows, int lane) const {
    const char* src = reinterpret_cast<const char*>(base);
    if (rows == TILE) {
#pragma unroll
      for (int j = 0; j < COPIES; ++j) tile::copy_1k(lds + 1024 * j, off[j], src);
    } else {
#pragma unroll
      for (int j = 0; j < COPIES; ++j) tile::copy_1k_ragged(lds + 1024 * j, offset(j, lane, rows), src);
    }
  }
  // Waits for every load of the wavefront, takes the tile; on return the stage may be filled again.
  static __device__ __forceinline__ void take(Rows<D>& k, const char* stage, int lane) {
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
      k.v[j] = *reinterpret_cast<const f32x4*>(stage + n * (D * 4) + (((4 * j + g) ^ n) << 4));
    wait_lgkmcnt0();
    __builtin_amdgcn_sched_barrier(0);
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

// Scores are kept as s * c and turned into probabilities 2^((s * c - reference) * up): c * up = sm_scale * log2 e with |c| at
// most 1 and `up` a power of two (1 for any ordinary scale), so that no finite score becomes infinite.  The running
// references start at LOWEST, below which there is no finite number: rows masked throughout to the type's lowest value
// have their maximum, and a score of -inf meets a finite reference.
constexpr float LOWEST = -3.402823466e38f;
struct Exponent {
  float c, up;
  __device__ __forceinline__ explicit Exponent(float sm_scale) : c(sm_scale * kLog2e), up(1.f) {
    if (fabsf(c) > 1.f) {
      up = ldexpf(1.f, __builtin_amdgcn_frexp_expf(c));
      c = __builtin_amdgcn_frexp_mantf(c);
    }
  }
  __device__ __forceinline__ float operator()(float s, float reference) const { return fast_exp2((s - reference) * up); }
};

// Reductions over the four lane groups (lanes n, n + 16, n + 32, n + 48), in a fixed order: groups 0 and 1, 2 and 3, then the
// two.  Swaps of registers, not exchanges through LDS: those take a round trip each, and the lane numbers that they need, which
// the calibration kernel (held to 128 registers at d = 128) formed anew at the end of every block of keys.  One call for a
// scale, d = 128, LDS -> swaps: 40 pairs, 144 x 265 keys 14.5 -> 14.1 us, 64 pairs, 144 x 720 36.7 -> 35.1; d = 64, 16 pairs,
// 276 x 614 16.5 -> 15.8.  Same bits.
__device__ __forceinline__ float max_groups(float v) {
  float even, odd;
  split_rows(v, even, odd);
  return max_halves(fmaxf(even, odd));
}
__device__ __forceinline__ float sum_groups(float v) {
  float even, odd;
  split_rows(v, even, odd);
  return sum_halves(even + odd);
}
// The same over a * b, on the lanes of groups 0 and 2: their own products enter unrounded.
__device__ __forceinline__ float sum_groups_product(float a, float b) {
  float even, odd;
  split_rows(a * b, even, odd);
  return sum_halves(fmaf(a, b, odd));
}

}  // namespace f32m
}  // namespace heatkv
