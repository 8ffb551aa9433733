// Cache update after a layer has run at scale k (Sec. 3.3): the layer's per-head
// runs are rewritten into the form the next scale reads.  Every block of rows to
// move was fixed by the planner (the schedule is static), so the kernel is a
// descriptor-driven streaming copy: 16 bytes per lane, a row of 256 bytes is one
// coalesced access of 16 lanes, K and V arenas handled by the same workgroup.
#include "copy_rows.h"
#include "device_util.h"
#include "kernels.h"

namespace heatkv {

namespace {

// PARTS workgroups share a descriptor.
template <int PARTS>
__global__ __launch_bounds__(256) void append_kernel(CopyParams p) {
  copy_rows_block(p, blockIdx.x, blockIdx.y, PARTS == 1 ? 0 : blockIdx.z, PARTS);
}

}  // namespace

hipError_t launch_append(const AppendArgs& a, hipStream_t stream) {
  if (a.ndesc <= 0) return hipSuccess;
  if (a.row_bytes % 16 != 0) return hipErrorInvalidValue;
  CopyParams p{};
  p.chunks_per_row = a.row_bytes / 16;
  p.kv_fp8 = a.kv_fp8 ? 1 : 0;
  p.H = a.H;
  p.t_k = a.t_k;
  p.arena_tokens = a.arena_tokens;
  p.descs = a.descs;
  p.k_new = static_cast<const uint4*>(a.k_new);
  p.v_new = static_cast<const uint4*>(a.v_new);
  p.k_arena = static_cast<uint4*>(a.k_arena);
  p.v_arena = static_cast<uint4*>(a.v_arena);
  // Four workgroups share a descriptor of rows of 256 bytes and more: one alone runs up to four rounds of loads and stores
  // one behind the other (the last chunks of a descriptor, and rows converted to 8-bit codes, come 256 at a time), and a
  // launch is only a few such rounds long.  Two serving layers (16 heads, d = 128, batch 32): 435 -> 423 us an image, with
  // 8-bit rows 291 -> 276; six layers of 32 heads at batch 2: 337 -> 322.  A descriptor of 128-byte rows is one round:
  // d = 64, 256 pairs, 130 us either way.  Their number is a constant of the kernel: read from the launch it costs every
  // small launch 0.1-0.2 us.
  if (p.chunks_per_row >= 16)
    hipLaunchKernelGGL(append_kernel<4>, dim3(a.ndesc, a.batch, 4), dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(append_kernel<1>, dim3(a.ndesc, a.batch), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace heatkv
