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
  // Workgroups with blockIdx.x >= attend_blocks run the fused cache update (copy descriptor, batch entry).
  // They sit at the end of the grid on purpose: there they fill the slots that the last attention workgroups
  // leave one by one.  Spread through the grid instead, their memory traffic lengthened the latency of the
  // attention workgroups' tile fetches and the launch became up to 1.4x slower.
  int attend_blocks;
  int ndesc;
  CopyParams copy;
};

// attend_f32.hip; `p` filled in except for the split into workgroups, copy_blocks = workgroups of the fused update.
hipError_t launch_attend_f32(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream);

}  // namespace heatkv
