// Kernel arguments of the attention kernels (bf16: attend.hip, attend_short.hip; fp32: attend_f32.hip, attend_f32_split.hip).
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

// What an attention workgroup works on: query tile qt of a (batch row, head) pair, and the head's run in the arena.
struct Task {
  int h, b, qt, run_row, run_len;
};
// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  All query tiles of a pair read the same K/V, so
// they have ids on one XCD; pairs come by decreasing run length and are dealt to the XCDs back and forth (0..7, 7..0, ...),
// which balances them.  False: a pair past the end (pairs are padded to a multiple of 8).
__device__ __forceinline__ bool find_task(const AttendParams& p, Task& t) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int turn = fast_div(slot, p.n_qtiles, p.div_qtiles);
  const int pair = turn * 8 + ((turn & 1) ? 7 - xcd : xcd);
  if (pair >= p.H * p.batch) return false;
  t.qt = slot - turn * p.n_qtiles;
  const int rank = fast_div(pair, p.batch, p.div_batch);
  t.b = pair - rank * p.batch;
  if (p.uniform_len >= 0) {
    t.h = rank;
    t.run_len = p.uniform_len;
    t.run_row = p.uniform_row0 + t.h * p.uniform_len;
  } else {
    // One 16-byte record: head, first row and length of its run.  Read as constant memory, i.e. by a scalar load: what
    // follows from it (tile addresses, descriptors) is then known to be wavefront-uniform.
    const auto* hw = (const __attribute__((address_space(4))) HeadWork*)(p.work) + rank;
    t.h = hw->head;
    t.run_len = hw->run_len;
    t.run_row = hw->run_row;
  }
  return true;
}

constexpr int TWO_STREAM_MIN_TOKENS = 384;  // two key streams per workgroup (attend.hip): shorter walks gain nothing

// attend_f32.hip and attend_short.hip (bf16, native cache rows); `p` filled in except for the split into workgroups,
// max_len = longest run, copy_blocks = workgroups of the fused update.
hipError_t launch_attend_f32(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream);
bool attend_short_fits(const AttendParams& p, int d, int max_len, unsigned copy_blocks);
hipError_t launch_attend_short(AttendParams p, int d, int max_len, unsigned copy_blocks, hipStream_t stream);
hipError_t attend_short_prepare();  // once per device
// attend_f32_split.hip: the same for fp32 launches of many queries and keys.
hipError_t launch_attend_f32_split(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream);
hipError_t attend_f32_split_prepare();  // once per device

}  // namespace heatkv
