// Next-scale attention over the ragged per-head KV cache, fp32 (attend.hip describes the path).
//
// Matrix-core kernel in full fp32.  A workgroup takes 16 queries; its four wavefronts split the keys (tiles of 16,
// dealt round robin, current scale first, then the head's retained run), each with a running reference, row sums and
// accumulators of its own, and are merged through LDS at the end.  fp32 problems are small (reference outputs,
// checks): a launch rarely has more than a few hundred query tiles, so the split over keys is what fills the chip.
//
// S^T = K Q^T leaves lane (n, g) with keys 4 g .. 4 g + 3 of query n, which is the B operand of O^T += V^T P^T as it
// stands: MFMA step r of a tile takes the keys 4 g + r.  V^T is the A operand; row n of accumulator block 4 j + i
// stands for column 64 j + 4 n + i, so that 16 lanes read 64 consecutive floats of a V row, 16 bytes each.
//
// Bound: the matrix pipe plus the vector instructions that do not overlap with it (f32_mfma.h) where a launch fills the
// chip (128 pairs x 400 queries x 800 keys, d = 128: 204 us = 103 TFLOP/s of the 151 a large fp32 matrix product reaches
// here; d = 64, 784 x 1384: 315 us = 113), the distribution of a few workgroups per compute unit below that (16 pairs,
// 625 + 500 keys: 70 us = 82 TFLOP/s).  The vector-ALU kernel that this one replaced fed its FMAs from LDS and reached 7
// TFLOP/s (the 625-query layer of a pruned image: 334 -> 62 us).  On the first shape, before scores and values had their
// full range (200 us then): keys straight into registers instead of through the stage 221 us with the compiler's 64-bit
// vector addresses, 208 us with scalar ones.  Eight wavefronts per workgroup, or 32 queries per workgroup (half the loads
// per MFMA): 0-15 % slower at every size, the first for the longer merge, the second for the coarser distribution and one
// wavefront less per SIMD.
#include "attend_params.h"
#include "device_util.h"
#include "f32_mfma.h"
#include "f32_split.h"
#include "kernels.h"

namespace heatkv {

namespace {

constexpr int NW = 4;  // wavefronts of a workgroup

template <int D>
__global__ __launch_bounds__(64 * NW) void attend_f32_kernel(AttendParams p) {
  constexpr int T = f32m::TILE;
  constexpr int NB = D / 16;    // accumulator blocks of 16 columns
  constexpr int PITCH = D + 4;  // floats per row of a parked output tile
  using Stage = f32m::KeyStage<D>;
  static_assert(T * PITCH * 4 >= Stage::BYTES, "the parked output tiles take the place of the key stages");
  __shared__ __attribute__((aligned(1024))) float park[NW][T][PITCH];
  __shared__ float part_m[NW][T], part_l[NW][T];

  touch_params(p);
  if (static_cast<int>(blockIdx.x) >= p.attend_blocks) {  // fused append: a plain row copy
    const int j = blockIdx.x - p.attend_blocks;
    copy_rows_block(p.copy, j % p.ndesc, j / p.ndesc);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Task task;
  if (!find_task(p, task)) return;
  const int h = task.h, b = task.b, qt = task.qt, n_prior = task.run_len, run_row = task.run_row;
  const int t_k = p.t_k;
  const long long cur_off = (static_cast<long long>(b) * p.H + h) * t_k * D;
  const long long run_off = (static_cast<long long>(b) * p.arena_tokens + run_row) * D;
  const float* k_cur = static_cast<const float*>(p.k_cur) + cur_off;
  const float* v_cur = static_cast<const float*>(p.v_cur) + cur_off;
  const float* k_prior = static_cast<const float*>(p.k_arena) + run_off;
  const float* v_prior = static_cast<const float*>(p.v_arena) + run_off;
  const long long q_off = cur_off + static_cast<long long>(qt) * T * D;
  const int q_rows = min(t_k - qt * T, T);

  const int tiles_cur = (t_k + T - 1) / T;
  const int tiles_all = tiles_cur + (n_prior + T - 1) / T;
  struct Tile {
    bool prior;
    long long first;  // element offset of its first row in the segment
    int rows;         // valid rows, 1..16
  };
  auto tile_of = [&](int it) {
    const bool prior = it >= tiles_cur;
    const int local = prior ? it - tiles_cur : it;
    return Tile{prior, static_cast<long long>(local) * (T * D), min((prior ? n_prior : t_k) - local * T, T)};
  };

  const char* stage = reinterpret_cast<const char*>(&park[0][0][0]) + wave * Stage::BYTES;
  const Stage keys(stage, lane);
  f32m::Rows<D> q, k;
  auto fetch = [&](int it) {
    const Tile t = tile_of(it);
    keys.fill((t.prior ? k_prior : k_cur) + t.first, t.rows, lane);
  };
  q.load(static_cast<const float*>(p.q) + q_off, q_rows, lane);
  if (wave < tiles_all) fetch(wave);

  f32x4 o[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // The reference m of a query is common to its four lanes and only raised when a score's exponent exceeds it by more than
  // 8: the accumulators are rescaled a few times per row.  Probabilities are taken 2^-8 times, at most 1, so that values
  // up to the type's largest over the number of keys can be summed.
  const f32m::Exponent prob(p.sm_scale);
  const float slack = 8.f / prob.up;
  float m = f32m::LOWEST, l = 0.f;

  for (int it = wave; it < tiles_all; it += NW) {
    const Tile t = tile_of(it);
    const f32m::GlobalBytes vb = f32m::scalar_base((t.prior ? v_prior : v_cur) + t.first);
    // K of the tile out of the stage, the copy of the next one into it, V: the waits for V then also cover that copy,
    // which is older, and the next step starts without waiting.
    Stage::take(k, stage, lane);
    if (it + NW < tiles_all) fetch(it + NW);
    f32x4 v[4][NB / 4];  // rows 4 g + r, columns 64 j + 4 n .. + 3
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned off = (min(4 * g + r, t.rows - 1) * D + 4 * n) * 4;
#pragma unroll
      for (int j = 0; j < NB / 4; ++j) v[r][j] = f32m::load16(vb, off + 256 * j);
    }
    f32x4 s = f32m::scores<D>(k, q);
    s *= prob.c;
    if (t.rows < T) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * g + r >= t.rows) {  // V too: these lanes hold the last valid row again, and 0 x inf is NaN
          s[r] = -INFINITY;
#pragma unroll
          for (int j = 0; j < NB / 4; ++j) v[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    const float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    if (__any(mx > m + slack)) {
      const float m_new = fmaxf(m, f32m::max_groups(mx));
      const float alpha = prob(m, m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < NB; ++i) o[i] *= alpha;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = prob(s[r], m) * 0x1p-8f;
    l += (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < NB; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][i / 4][i % 4], s[r], o[i], 0, 0, 0);
  }

  // Merge: every wavefront brings its accumulators to the common reference and divides by the common row sum; the
  // parked tiles are then added in wavefront order.  A wavefront without a tile has the lowest reference: factor 0.
  __syncthreads();  // every wavefront has taken its last tile
  l = f32m::sum_groups(l);
  if (g == 0) {
    part_m[wave][n] = m;
    part_l[wave][n] = l;
  }
  __syncthreads();
  float m_all = part_m[0][n], l_all = 0.f;
#pragma unroll
  for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, part_m[w][n]);
#pragma unroll
  for (int w = 0; w < NW; ++w) l_all += part_l[w][n] * prob(part_m[w][n], m_all);
  const float f = prob(m, m_all) / l_all;
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int j = 0; j < NB / 4; ++j) {  // lane (n, g) holds columns 64 j + 16 g + 4 r + i of query n
      const f32x4 x = {o[4 * j][r], o[4 * j + 1][r], o[4 * j + 2][r], o[4 * j + 3][r]};
      *reinterpret_cast<f32x4*>(&park[wave][n][64 * j + 16 * g + 4 * r]) = x * f;
    }
  __syncthreads();
  float* out = static_cast<float*>(p.out) + q_off;
  for (int e = tid; e < q_rows * (D / 4); e += 64 * NW) {
    const int row = e / (D / 4), col = e % (D / 4) * 4;
    f32x4 x = *reinterpret_cast<const f32x4*>(&park[0][row][col]);
#pragma unroll
    for (int w = 1; w < NW; ++w) x += *reinterpret_cast<const f32x4*>(&park[w][row][col]);
    *reinterpret_cast<f32x4*>(out + row * D + col) = x;
  }
}

}  // namespace

hipError_t launch_attend_f32(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream) {
  const unsigned long long all = (unsigned long long)((p.H * p.batch + 7) / 8 * 8);
  if ((d == 64 || d == 128) && f32s::pays(d, p.t_k, (p.t_k + 15) / 16 * all, (p.t_k + 31) / 32 * all, p.sm_scale))
    return launch_attend_f32_split(p, d, copy_blocks, stream);
  p.n_qtiles = (p.t_k + f32m::TILE - 1) / f32m::TILE;
  const unsigned pairs8 = (unsigned(p.H) * p.batch + 7) / 8 * 8;  // padded so that id % 8 is the XCD
  p.attend_blocks = int(unsigned(p.n_qtiles) * pairs8);
  p.div_qtiles = reciprocal(p.attend_blocks, p.n_qtiles);
  p.div_batch = reciprocal(pairs8, p.batch);
  const dim3 grid(unsigned(p.attend_blocks) + copy_blocks), block(64 * NW);
  if (d == 64)
    hipLaunchKernelGGL(attend_f32_kernel<64>, grid, block, 0, stream, p);
  else if (d == 128)
    hipLaunchKernelGGL(attend_f32_kernel<128>, grid, block, 0, stream, p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace heatkv
