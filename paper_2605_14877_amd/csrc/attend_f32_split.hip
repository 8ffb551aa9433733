// Next-scale attention over the ragged per-head KV cache, fp32, for launches of many queries and keys (attend.hip describes
// the path, f32_split.h the arithmetic and when this kernel is taken; attend_f32.hip is the other one).
//
// A workgroup takes 32 queries; its eight wavefronts split the keys (blocks of 32, dealt round robin, current scale first,
// then the head's retained run), each with a reference, row sums and accumulators of its own, and are merged through LDS
// at the end.  Keys go through an LDS stage per wavefront, values straight into registers: a lane's eight keys of four
// (d = 64: two) neighbouring columns are the A operands of as many accumulator blocks.  The parts of the queries lie in LDS,
// those of keys, values and probabilities are formed in registers, between the products of the block before them: a
// wavefront issues in order.
//
// Bound: vector instructions, 44 of them for the six products of a step (48 with the magnitudes), which take 75 to 80 clocks a
// product when a wavefront has the SIMD to itself and about half of that per product when two share it.  fp32 instructions ->
// this kernel, d = 128: 16 pairs, 784 queries x up to 2194 keys 129 -> 105 us, 8 pairs 529 x 2160 83 -> 60, 256 pairs 625 x 2525
// 1221 -> 1039.  Error against 64 bits (norm) on the same inputs, 18 kinds of them: 0.65 to 0.72 times that of the fp32
// instructions, 1.8-2.2e-7 for 2.5-3.3e-7 on N(0,1) operands, 3.7-4.9e-7 for 5.2-7.1e-7 on scores four times as large.
#include <atomic>

#include "attend_params.h"
#include "device_util.h"
#include "f32_mfma.h"
#include "f32_split.h"
#include "tile_lds.h"

namespace heatkv {

namespace {

constexpr int NW = 8;  // wavefronts of a workgroup
constexpr int BQ = 32, BK = 32;  // queries of a workgroup, keys of a block

extern __shared__ __attribute__((aligned(1024))) char f32_lds[];

template <int D>
struct F32Lds {
  static constexpr int ROW = 4 * D, STAGE = BK * ROW;  // one key row, the keys of a block
  static constexpr int Q = NW * STAGE;                 // [part][step][lane] 16 bytes: the query rows in three bf16 parts
  static constexpr int M = Q + 3 * (D / 16) * 1024;    // references and row sums for the merge, [wavefront][query]
  static constexpr int L = M + NW * BQ * 4;
  static constexpr int BIG = L + NW * BQ * 4;          // per wavefront: the query elements that it has seen are too large
  static constexpr int BYTES = BIG + NW * 4;
};

template <int D>
__global__ __launch_bounds__(64 * NW) void attend_f32_split_kernel(AttendParams p) {
  using Lds = F32Lds<D>;
  constexpr int NK = D / 16;   // MFMA steps of a score block
  constexpr int NV = D / 32;   // accumulator blocks; block i holds the columns NV m + i (m = 0..31)
  constexpr int ROW = Lds::ROW, CPR = D / 4;  // bytes, 16-byte chunks of a row
  constexpr int COPIES = Lds::STAGE / 1024;

  touch_params(p);
  if (static_cast<int>(blockIdx.x) >= p.attend_blocks) {  // fused append: a plain row copy
    const int j = blockIdx.x - p.attend_blocks;
    copy_rows_block(p.copy, j % p.ndesc, j / p.ndesc, threadIdx.x >> 8, NW / 4);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Task task;
  if (!find_task(p, task)) return;
  const int t_k = p.t_k, n_prior = task.run_len;
  const long long cur_off = (static_cast<long long>(task.b) * p.H + task.h) * t_k * D;
  const long long run_off = (static_cast<long long>(task.b) * p.arena_tokens + task.run_row) * D;
  const float* k_cur = static_cast<const float*>(p.k_cur) + cur_off;
  const float* v_cur = static_cast<const float*>(p.v_cur) + cur_off;
  const float* k_prior = static_cast<const float*>(p.k_arena) + run_off;
  const float* v_prior = static_cast<const float*>(p.v_arena) + run_off;
  const long long q_off = cur_off + static_cast<long long>(task.qt) * BQ * D;
  const int q_rows = min(t_k - task.qt * BQ, BQ);

  const int blocks_cur = (t_k + BK - 1) / BK;
  const int blocks_all = blocks_cur + (n_prior + BK - 1) / BK;
  struct Block {
    bool prior;
    int local, rows;  // number inside its segment, valid rows from its first one on (32 and more: all)
  };
  auto block_of = [&](int it) {
    const bool prior = it >= blocks_cur;
    const int local = prior ? it - blocks_cur : it;
    return Block{prior, local, (prior ? n_prior : t_k) - local * BK};
  };

  // Key rows of a block to the wavefront's stage, the 16-byte chunks of a row XORed with the row number (f32_mfma.h); rows
  // past the end are zeros.
  char* const stage = f32_lds + wave * Lds::STAGE;
  const unsigned stage_lds = static_cast<unsigned>(
      reinterpret_cast<unsigned long long>((__attribute__((address_space(3))) char*)(&f32_lds[0]))) + wave * Lds::STAGE;
  constexpr int ROWS = 64 / CPR;  // of a copy
  auto fetch = [&](int it) {
    const Block t = block_of(it);
    const tile::Descriptor src = tile::tile_descriptor<ROW>(
        reinterpret_cast<const char*>((t.prior ? k_prior : k_cur) + static_cast<long long>(t.local) * (BK * D)), t.rows);
    // Row ROWS i + b, chunk c ^ row = (c ^ b) ^ ROWS i.  Formed anew for every block: there are no registers to keep it in.
    const int b = lane / CPR;
    int off = b * ROW + (((lane & (CPR - 1)) ^ b) << 4);
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int i = 0; i < COPIES; ++i)
      tile::copy_1k_checked(stage_lds, i * 1024, off ^ ((ROWS * i & 15) << 4), src, i * 1024);
  };
  if (wave < blocks_all) fetch(wave);

  // The query rows in three parts, as the B operand: wavefront `step` splits the elements 16 step + 8 hl .. + 7 of row n.
  const float* const q_row = static_cast<const float*>(p.q) + q_off + min(n, q_rows - 1) * D + 8 * hl;
  auto load_q = [&](int step, float (&x)[8]) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(q_row + 16 * step), b = *reinterpret_cast<const f32x4*>(q_row + 16 * step + 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = a[j];
      x[4 + j] = b[j];
    }
  };
  float q_most = 0.f;
  if (wave < NK) {
    float x[8];
    load_q(wave, x);
    q_most = f32s::magnitude(0.f, x);
    f32s::Parts parts;
    f32s::split(parts, x);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      *reinterpret_cast<bf16x8*>(f32_lds + Lds::Q + (i * NK + wave) * 1024 + lane * 16) = parts.part(i);
  }
  int* const big = reinterpret_cast<int*>(f32_lds + Lds::BIG);
  if (lane == 0) big[wave] = 0;
  if (__any(q_most > f32s::LARGEST) && lane == 0) big[wave] = 1;
  __syncthreads();
  int q_big = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) q_big |= big[w];
  q_big = __builtin_amdgcn_readfirstlane(q_big);

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  // The reference m of a query is common to its two lanes and only raised when a score's exponent exceeds it by more than
  // 8: the accumulators are rescaled a few times per row.  Probabilities are taken 2^-8 times, at most 1, so that values
  // up to the type's largest over the number of keys can be summed.
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  const f32m::Exponent prob(p.sm_scale);
  const float slack = 8.f / prob.up;
  float m = f32m::LOWEST, l = 0.f;

  for (int it = wave; it < blocks_all; it += NW) {
    const Block t = block_of(it);
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    // Values of 16 keys: element j of lane (n, hl) and chunk c is key 16 c + 8 (j / 4) + 4 hl + j % 4 (the order of the
    // probabilities below), columns NV n ..; rows past the end are zeros.
    const auto v_rows = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>((t.prior ? v_prior : v_cur) + static_cast<long long>(t.local) * (BK * D)), 0,
        min(t.rows, BK) * ROW, 0x00020000);
    auto load_v = [&](int c, float (&v)[8][NV]) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int off = 4 * hl * ROW + n * (NV * 4), at = (16 * c + 8 * (j >> 2) + (j & 3)) * ROW;
        if constexpr (NV == 4) {
          const auto x = __builtin_amdgcn_raw_buffer_load_b128(v_rows, off, at, 0);
#pragma unroll
          for (int i = 0; i < NV; ++i) v[j][i] = __uint_as_float(x[i]);
        } else {
          const auto x = __builtin_amdgcn_raw_buffer_load_b64(v_rows, off, at, 0);
#pragma unroll
          for (int i = 0; i < NV; ++i) v[j][i] = __uint_as_float(x[i]);
        }
      }
    };
    float v0[8][NV], v1[8][NV];
    load_v(0, v0);
    // Chunks 4 step + 2 hl and the next one of row n, XORed with the row: address bits 4 to 8, in which the row's own
    // address has no ones.  Formed anew for every block, like the copies' offsets.
    unsigned k_at = stage_lds + n * ROW + (((2 * hl) ^ (n & 15)) << 4);
    asm volatile("" : "+v"(k_at));
    auto load_k = [&](int step, float (&x)[8]) {
      typedef const __attribute__((address_space(3))) f32x4* LdsChunk;
      const f32x4 a = *(LdsChunk)(k_at ^ (step << 6)), b = *(LdsChunk)(k_at ^ (step << 6) ^ 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[j] = a[j];
        x[4 + j] = b[j];
      }
    };
    f32x16 s, small;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = small[r] = 0.f;
    float k_most = 0.f;
    // In the slots between the matrix instructions of a step: the query parts of its successor, the split of its successor's keys,
    // the keys after that.  (In one piece, the split in front of the products it feeds, a wavefront waits for either.)
    float x[2][8];
    f32s::Parts kp[2], qp;
    auto read_q = [&](int step, int part) {
      qp.set(part, *reinterpret_cast<const bf16x8*>(f32_lds + Lds::Q + (part * NK + step) * 1024 + lane * 16));
    };
    load_k(0, x[0]);
#pragma unroll
    for (int i = 2; i >= 0; --i) read_q(0, i);
    load_k(1, x[1]);
    k_most = f32s::magnitude(k_most, x[0]);
    f32s::split(kp[0], x[0]);
#pragma unroll
    for (int step = 0; step < NK; ++step)
#pragma unroll
      for (int m = 0; m < f32s::PRODUCTS; ++m) {
        fence();
        f32s::add_product(m, small, s, kp[step & 1], qp);
        fence();
        if (step + 1 < NK && (m == 0 || m == 2 || m == 5)) read_q(step + 1, m == 0 ? 2 : m == 2 ? 1 : 0);
        if (m == 0 && step + 2 < NK) load_k(step + 2, x[step & 1]);
        if (step + 1 < NK) {
          if (m == 0) k_most = f32s::magnitude(k_most, x[(step + 1) & 1]);
          f32s::split_piece(kp[(step + 1) & 1], x[(step + 1) & 1], m);
        }
      }
    fence();
    if (q_big || __any(k_most > f32s::LARGEST)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = small[r] = 0.f;
#pragma unroll 1
      for (int step = 0; step < NK; ++step) {
        float y[8], z[8];
        load_k(step, y);
        load_q(step, z);
        f32s::add_f32(s, y, z);
      }
    }
    wait_lgkmcnt0();
    wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
    if (it + NW < blocks_all) fetch(it + NW);
    load_v(1, v1);  // the wait for these covers the copies, which are older
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = (s[r] + small[r]) * prob.c;
    if (t.rows < BK) tile::mask_block(t.rows, hl, s);
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    if (__any(mx > m + slack)) {
      const float m_new = fmaxf(m, max_halves(mx));
      const float alpha = prob(m, m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < NV; ++i) o[i] *= alpha;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = prob(s[r], m) * 0x1p-8f;
    {
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[r & 3] += s[r];
      l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    }
    // The same with the split of the next accumulator block's values between the products of one.
    float pr[2][8];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) pr[c][j] = s[8 * c + j];
    f32s::Parts pp[2], vp[2];
    auto accumulate = [&](int c, const float (&v)[8][NV]) {
      // Operands that have exact parts, neither too large nor too small (f32_split.h).  Zeros are told from tiny numbers only
      // where there is one of either (16 pairs, 625 queries x up to 1139 keys: 52.8 us without the lower limit, 54.0 with it, 55.8
      // with a column of zeros).
      float most = 0.f, least = pr[c][0];
#pragma unroll
      for (int j = 0; j < 8; j += 2) least = fminf(least, fminf(pr[c][j], pr[c][j + 1]));
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < NV; i += 2) {
          most = fmaxf(most, fmaxf(fabsf(v[j][i]), fabsf(v[j][i + 1])));
          least = fminf(least, fminf(fabsf(v[j][i]), fabsf(v[j][i + 1])));
        }
      bool parts = !__any(most > f32s::LARGEST || least < f32s::SMALLEST);
      if (!parts && !__any(most > f32s::LARGEST)) {  // zeros (rows past the end, masked keys) have parts
        unsigned lowest = f32s::above_zero(pr[c][0]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          lowest = min(lowest, f32s::above_zero(pr[c][j]));
#pragma unroll
          for (int i = 0; i < NV; ++i) lowest = min(lowest, f32s::above_zero(v[j][i]));
        }
        parts = !__any(lowest < f32s::above_zero(f32s::SMALLEST));
      }
      if (parts) {
        float y[2][8];
        auto take = [&](int blk) {
#pragma unroll
          for (int j = 0; j < 8; ++j) y[blk & 1][j] = v[j][blk];
        };
        take(0);
        f32s::split(pp[c], pr[c]);
        f32s::split(vp[0], y[0]);
#pragma unroll
        for (int blk = 0; blk < NV; ++blk) {
          if (blk + 1 < NV) take(blk + 1);
#pragma unroll
          for (int m = 0; m < f32s::PRODUCTS; ++m) {
            fence();
            f32s::add_product(m, o[blk], o[blk], vp[blk & 1], pp[c]);
            fence();
            if (blk + 1 < NV) f32s::split_piece(vp[(blk + 1) & 1], y[(blk + 1) & 1], m);
          }
        }
        fence();
      } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          float y[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) y[j] = v[j][i];
          f32s::add_f32(o[i], y, pr[c]);
        }
      }
    };
    accumulate(0, v0);
    accumulate(1, v1);
  }

  // Merge: every wavefront brings its accumulators to the common reference and divides by the common row sum; the
  // parked tiles (in the place of the key stages) are then added in wavefront order.  A wavefront without a block has the
  // lowest reference: factor 0.
  float* const part_m = reinterpret_cast<float*>(f32_lds + Lds::M);
  float* const part_l = reinterpret_cast<float*>(f32_lds + Lds::L);
  l = sum_halves(l);
  if (hl == 0) {
    part_m[wave * BQ + n] = m;
    part_l[wave * BQ + n] = l;
  }
  __syncthreads();
  float m_all = part_m[n], l_all = 0.f;
#pragma unroll
  for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, part_m[w * BQ + n]);
#pragma unroll
  for (int w = 0; w < NW; ++w) l_all += part_l[w * BQ + n] * prob(part_m[w * BQ + n], m_all);
  const float f = prob(m, m_all) / l_all;
  // Register r of block i of lane (n, hl) is column NV (8 (r / 4) + 4 hl + r % 4) + i of query n.  Rows are XORed like the
  // stages, in units of NV floats.
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int at = 8 * (r >> 2) + 4 * hl + (r & 3);
    float* dst = reinterpret_cast<float*>(stage) + n * D + ((at ^ n) * NV);
#pragma unroll
    for (int i = 0; i < NV; ++i) dst[i] = o[i][r] * f;
  }
  __syncthreads();
  float* out = static_cast<float*>(p.out) + q_off;
  for (int e = tid; e < q_rows * 32; e += 64 * NW) {
    const int row = e >> 5, at = e & 31;
    float x[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) x[i] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* src = reinterpret_cast<const float*>(f32_lds + w * Lds::STAGE) + row * D + ((at ^ row) * NV);
#pragma unroll
      for (int i = 0; i < NV; ++i) x[i] = w == 0 ? src[i] : x[i] + src[i];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) out[row * D + at * NV + i] = x[i];
  }
}

}  // namespace

// More than 64 KB of dynamic LDS needs the function attribute raised, once per device.
hipError_t attend_f32_split_prepare() {
  static std::atomic<unsigned long long> done{0};  // one bit per device ordinal below 64
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 64 && (done.load(std::memory_order_acquire) >> dev & 1)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_f32_split_kernel<64>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, F32Lds<64>::BYTES);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_f32_split_kernel<128>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, F32Lds<128>::BYTES);
  if (e == hipSuccess && dev >= 0 && dev < 64) done.fetch_or(1ull << dev, std::memory_order_release);
  return e;
}

hipError_t launch_attend_f32_split(AttendParams p, int d, unsigned copy_blocks, hipStream_t stream) {
  const hipError_t e = attend_f32_split_prepare();
  if (e != hipSuccess) return e;
  p.n_qtiles = (p.t_k + BQ - 1) / BQ;
  const unsigned pairs8 = (unsigned(p.H) * p.batch + 7) / 8 * 8;  // padded so that id % 8 is the XCD
  p.attend_blocks = int(unsigned(p.n_qtiles) * pairs8);
  p.div_qtiles = reciprocal(p.attend_blocks, p.n_qtiles);
  p.div_batch = reciprocal(pairs8, p.batch);
  const dim3 grid(unsigned(p.attend_blocks) + copy_blocks), block(64 * NW);
  if (d == 64)
    hipLaunchKernelGGL(attend_f32_split_kernel<64>, grid, block, F32Lds<64>::BYTES, stream, p);
  else
    hipLaunchKernelGGL(attend_f32_split_kernel<128>, grid, block, F32Lds<128>::BYTES, stream, p);
  return hipGetLastError();
}

}  // namespace heatkv
