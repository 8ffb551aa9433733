// Kernel arguments of the attention kernels (attend.hip: bf16, attend_f32.hip: fp32).
#pragma once

#include "copy_rows.h"
#include "plan.h"

namespace heatkv {

struct AttendParams {
  int H, batch, t_k;
  long long arena_tokens;
  const HeadWork* work;
  // uniform_len >= 0: every head of the layer holds a run of that many rows, head h's run starts at row
  // uniform_row0 + h * uniform_len, and (batch row, head) pairs are taken in index order: a workgroup then knows
  // all its addresses from its id and the kernel arguments, and its first fetches do not wait for a table read.
  int uniform_len, uniform_row0;
  const void *q, *k_cur, *v_cur, *k_arena, *v_arena;
  void* out;
  float sm_scale;
  int n_qtiles;
  unsigned div_qtiles, div_batch;  // reciprocals for fast_div, see reciprocal()
  // Workgroups with blockIdx.x >= attend_blocks run the fused cache update (copy descriptor, batch entry).
  // They sit at the end of the grid on purpose: there they fill the slots that the last attention workgroups
  // leave one by one.  Spread through the grid instead, their memory traffic lengthened the latency of the
  // attention workgroups' tile fetches and the launch became up to 1.4x slower.
  int attend_blocks;
  int ndesc;
  CopyParams copy;
};

// n / d for 0 <= n <= n_max, with a reciprocal from the host: exact as long as n_max * d < 2^32 (reciprocal() gives 0
// otherwise, and the division is carried out).  A workgroup divides twice before its first fetch, 25 dependent
// instructions each time.
inline unsigned reciprocal(unsigned long long n_max, unsigned d) {
  return d > 1 && n_max * d < (1ull << 32) ? static_cast<unsigned>((1ull << 32) / d + 1) : 0;
}
__device__ __forceinline__ int fast_div(int n, int d, unsigned recip) {
  return recip ? static_cast<int>(__umulhi(static_cast<unsigned>(n), recip)) : d == 1 ? n : n / d;
}

// The arguments that a workgroup needs before its first fetch, asked for together: left to itself the compiler reads
// them where they are used, three scalar-cache misses one after the other.
__device__ __forceinline__ void touch_params(const AttendParams& p) {
  asm volatile("; kernel arguments" ::"s"(p.H), "s"(p.arena_tokens), "s"(p.work), "s"(p.uniform_len), "s"(p.q), "s"(p.k_cur),
               "s"(p.v_cur), "s"(p.k_arena), "s"(p.v_arena), "s"(p.out), "s"(p.sm_scale), "s"(p.attend_blocks));
}

// attend_f32.hip; `p` filled in except for the split into workgroups, copy_blocks = workgroups of the fused update.
hipError_t launch_attend_f32(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream);

}  // namespace heatkv
