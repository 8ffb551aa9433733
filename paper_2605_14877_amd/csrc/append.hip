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
  // Four workgroups share a descriptor where one alone would run several rounds of loads and stores one behind the other
  // (whole groups of 1024 chunks are a round, the rest and rows converted to 8-bit codes come 256 chunks at a time: 127
  // rows of 256 bytes are five rounds) and the launch does not fill the chip: up to about 2048 workgroups are resident at
  // once.  Whole images: two serving layers (16 heads, d = 128, batch 32, 20x) 437 -> 428 us, with 8-bit rows 295 -> 282;
  // six layers of 32 heads, batch 2, 338 -> 323, with 8-bit rows 366 -> 288.  Single launches, one against four: 1536
  // descriptors of 88 rows 19.5 -> 18.3 us, 2304 of 102 rows 52.3 -> 52.3, 3856 of 124 rows 72.4 -> 75.4, 8448 of 125 rows
  // 196 -> 208; 8-bit rows (half the bytes, one chunk per lane and round) 4608 of 102 rows 61.6 -> 59.9, 7712 of 124 rows
  // 86 -> 89.6; one round of work on average: 1024 of 11 rows 3.3 -> 4.1, 512 2.6 -> 2.9, 256 and fewer no dearer, and there
  // the long ones among short ones count (the 8-bit images at batch 2).  128-byte rows: 130 us an image either way (d = 64,
  // 256 pairs).  The number is a constant of the kernel: read from the launch it costs every small launch 0.1-0.2 us.
  const long long arena_chunks = a.kv_fp8 ? p.chunks_per_row / 2 : p.chunks_per_row;
  const long long descriptors = static_cast<long long>(a.ndesc) * a.batch, most = a.kv_fp8 ? 4608 : 2304;
  const bool several_rounds = a.rows * arena_chunks > 256ll * a.ndesc || descriptors <= 256;
  if (p.chunks_per_row >= 16 && several_rounds && descriptors <= most)
    hipLaunchKernelGGL(append_kernel<4>, dim3(a.ndesc, a.batch, 4), dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(append_kernel<1>, dim3(a.ndesc, a.batch), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace heatkv
