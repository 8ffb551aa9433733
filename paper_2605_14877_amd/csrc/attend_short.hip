// Next-scale attention over the ragged per-head KV cache, bf16, for launches that leave most of the chip idle when a
// wavefront walks all keys of its 32 queries alone (attend.hip describes the path, tile format and operand layouts).
//
// A workgroup takes 32 queries (d = 128) or two sets of 32 (d = 64) and walks the keys in rounds of two 64-row tiles.  The
// W = d / 32 wavefronts of a query set share a round's work twice over:
//   scores:  each takes its part of the 128 keys, S^T = K Q^T, and leaves its row maxima in LDS; every wavefront then
//            follows the running reference through the round's tiles, so that all of them agree on it;
//   P V:     the probabilities go through LDS, and each wavefront accumulates 32 of the d output columns over all keys.
// There is nothing to merge at the end, and every number is formed as in the one-wavefront walk (same reference, same order
// of the sums over keys): the outputs are the same, bit for bit.
//
// Bound: latency.  A launch of a few workgroups spends about 1700 cycles until its first keys are there (kernel arguments,
// one round trip to memory), 1100 in the scores, 900 in reference and probabilities, 500 to 1100 in P V (by the number of
// keys, of which only chunks of 16 with a valid one are copied and multiplied), 900 in the output, and 1.2 us outside the
// kernel; a wavefront that does all of it alone takes 2100 + 3300 + 1150 for the same.  A further round adds 3000 to 4000
// cycles, of which 1700 go to issuing its 64 copies of 1 KB, under the work of the round before.
#include <algorithm>

#include "attend_params.h"
#include "device_util.h"
#include "tile_lds.h"

namespace heatkv {

namespace {

extern __shared__ __attribute__((aligned(1024))) char short_lds[];

// STAGES = 1: walks of at most two tiles, one round.  STAGES = 2: any walk, the tiles of two rounds in LDS.
template <int D, int STAGES>
struct ShortLds {
  static constexpr int TILE_BYTES = tile::ROWS * 2 * D;
  static constexpr int SETS = 128 / D;                   // query sets of 32
  static constexpr int K = 0, V = STAGES * 2 * TILE_BYTES;  // [stage][two tiles]
  static constexpr int P = 2 * V;                        // [set][chunk of 16 keys][lane] 16 bytes; at first the query rows
  static constexpr int MX = P + SETS * 8 * 1024;         // [set][block of 32 keys][query] float
  static constexpr int BYTES = MX + SETS * 4 * 32 * 4;
};

template <int D, int STAGES>
__global__ __launch_bounds__(512, STAGES == 1 ? 4 : 2) void attend_short_kernel(AttendParams p) {
  static_assert(D == 128 || D == 64, "head dimension 128 or 64");
  using Lds = ShortLds<D, STAGES>;
  constexpr int BN = tile::ROWS, ROW_BYTES = 2 * D, TILE_BYTES = Lds::TILE_BYTES;
  constexpr int NK = D / 16;               // MFMA steps of a block of 32 keys
  constexpr int SETS = Lds::SETS, NW = 4, W = NW / SETS;  // query sets, computing wavefronts, those of a set
  constexpr int U = 4 / W;                 // blocks of 32 keys per wavefront and round
  constexpr int COPIES = TILE_BYTES / 1024, ROWS_PER_COPY = 1024 / ROW_BYTES;

  touch_params(p);
  if (static_cast<int>(blockIdx.x) >= p.attend_blocks) {  // fused append: a plain row copy
    const int j = blockIdx.x - p.attend_blocks;
    copy_rows_block(p.copy, j % p.ndesc, j / p.ndesc, threadIdx.x >> 8, 2);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hl = lane >> 5;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave_all & (NW - 1);
  Task task;
  if (!find_task(p, task)) return;
  const int t_k = p.t_k, n_prior = task.run_len;
  const long long cur_off = (static_cast<long long>(task.b) * p.H + task.h) * t_k * ROW_BYTES;
  const int block_row0 = task.qt * (32 * SETS);
  const int tiles_cur = (t_k + BN - 1) / BN;
  const int tiles_all = tiles_cur + (n_prior + BN - 1) / BN;
  const int rounds = STAGES == 1 ? 1 : (tiles_all + 1) / 2;
  // Rows of tile j from its first one to the end of its segment (current scale first, then the retained run); none past
  // the walk's end.
  auto rows_left = [&](int j) {
    return j < tiles_cur ? t_k - j * BN : j < tiles_all ? n_prior - (j - tiles_cur) * BN : 0;
  };

  // Four wavefronts copy, four compute: a wavefront is held up for some 100 cycles by each copy that it issues in a row.
  if (wave_all >= NW) {
    const long long run_off = (static_cast<long long>(task.b) * p.arena_tokens + task.run_row) * ROW_BYTES;
    const char* const k_cur = static_cast<const char*>(p.k_cur) + cur_off;
    const char* const v_cur = static_cast<const char*>(p.v_cur) + cur_off;
    const char* const k_prior = static_cast<const char*>(p.k_arena) + run_off;
    const char* const v_prior = static_cast<const char*>(p.v_arena) + run_off;
    const unsigned lds_wave = static_cast<unsigned>(reinterpret_cast<unsigned long long>(
                                  (__attribute__((address_space(3))) char*)(&short_lds[0]))) + wave * 1024;
    const int ld_off_k = tile::loader_off_k<ROW_BYTES>(wave, lane);
    const int ld_off_v = tile::loader_off_v<ROW_BYTES>(wave, lane);
    // This wavefront's share of the copies of the first `rows` rows of a tile with `left` valid ones, the others as zeros;
    // how many it issued.
    auto issue_rows = [&](const char* src, int left, int rows, int off, int dst) {
      const tile::Descriptor t = tile::tile_descriptor<ROW_BYTES>(src, left);
      int issued = 0;
#pragma unroll
      for (int i = 0; i < COPIES / NW; ++i)
        if ((i * NW + wave) * ROWS_PER_COPY < rows) {
          tile::copy_1k_checked(lds_wave + dst, i * (1024 * NW), off, t, i * (1024 * NW));
          ++issued;
        }
      return issued;
    };
    auto issue_round = [&](int r, int dst, int off, const char* cur, const char* prior) {
      int issued = 0;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int j = 2 * r + i;
        const int local = j < tiles_cur ? j : j - tiles_cur;
        const int left = rows_left(j);  // what the round reads: the chunks of 16 keys that have a valid one
        issued += issue_rows((j < tiles_cur ? cur : prior) + static_cast<long long>(local) * TILE_BYTES, left,
                             (left + 15) & ~15, off, dst + ((r & (STAGES - 1)) * 2 + i) * TILE_BYTES);
      }
      return issued;
    };
    auto issue_k = [&](int r) { return issue_round(r, Lds::K, ld_off_k, k_cur, k_prior); };
    auto issue_v = [&](int r) { return issue_round(r, Lds::V, ld_off_v, v_cur, v_prior); };

    // Query rows in the place of the probabilities, laid out as a K tile; rows past t_k are zeros (they must not raise the
    // reference of their set).
    issue_rows(static_cast<const char*>(p.q) + cur_off + static_cast<long long>(block_row0) * ROW_BYTES, t_k - block_row0,
               32 * SETS, ld_off_k, Lds::P);
    issue_k(0);
    wait_vmcnt<0>();
    __syncthreads();  // (1)
    issue_v(0);
    if (rounds > 1) issue_k(1);
    for (int r = 0;; ++r) {
      __syncthreads();  // (2) K(r) and V(r - 1) have been read
      int younger = 0;  // copies in flight that the wait leaves alone
      if (r + 1 < rounds) younger = issue_v(r + 1);
      if (r + 2 < rounds) younger += issue_k(r + 2);
      constexpr int MOST = 4 * COPIES / NW;  // V and K of two full tiles
      if (younger == MOST)
        wait_vmcnt<MOST>();
      else if (younger >= MOST / 2)
        wait_vmcnt<MOST / 2>();
      else
        wait_vmcnt<0>();
      __syncthreads();  // (3) V(r) and K(r + 1) are there
      if (r + 1 == rounds) return;
    }
  }

  const int set = wave / W, w = wave % W;
  const int q_row0 = block_row0 + 32 * set;
  const bool active = q_row0 < t_k;  // a set past the last query row only keeps the barriers
  int k_off[NK], v_off[D / 32];
  tile::reader_off_k<ROW_BYTES>(lane, k_off);
  tile::reader_off_v<ROW_BYTES>(lane, v_off);
  const float c = p.sm_scale * kLog2e;
  float m_run = lowest_reference(c), l_run = 0.f;
  constexpr float kSlack = 8.f;  // as in the one-wavefront walk
  const float slack_raw = kSlack / c;
  const bf16x2 ones = {static_cast<bf16_t>(1.f), static_cast<bf16_t>(1.f)};
  f32x16 o;
#pragma unroll
  for (int i = 0; i < 16; ++i) o[i] = 0.f;
  float* const mx_set = reinterpret_cast<float*>(short_lds + Lds::MX) + set * (4 * 32);
  char* const p_set = short_lds + Lds::P + set * (8 * 1024) + lane * 16;
  bf16x8 qreg[NK];
  f32x16 s[U];

  // Left to itself the compiler reads an operand, waits for it, uses it and reads the next one into the same registers.
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  // This wavefront's blocks of 32 keys of round r: scores, and their row maxima to LDS (-inf for a block without a key).
  auto scores = [&](int r) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int blk = w * U + u;
      const int left = rows_left(2 * r + (blk >> 1)) - 32 * (blk & 1);
      float mx = -INFINITY;
      if (left > 0) {
        const char* kt = short_lds + Lds::K + (r & (STAGES - 1)) * (2 * TILE_BYTES) + blk * (32 * ROW_BYTES);
        bf16x8 a[NK];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) a[ks] = *reinterpret_cast<const bf16x8*>(kt + k_off[ks]);
        fence();
#pragma unroll
        for (int i = 0; i < 16; ++i) s[u][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], qreg[ks], s[u], 0, 0, 0);
        if (left < 32) tile::mask_block(left, hl, s[u]);
        mx = s[u][0];
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[u][i]);
        mx = max_halves(mx);
      }
      if (hl == 0) mx_set[blk * 32 + n] = mx;
    }
  };
  // The reference through the round's two tiles; whether it was raised is the same for the whole wavefront.
  float alpha[2], reference[2];
  bool raised[2];
  auto follow_reference = [&] {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float mx = fmaxf(mx_set[(2 * i) * 32 + n], mx_set[(2 * i + 1) * 32 + n]);
      raised[i] = __any(mx > m_run + slack_raw);
      if (raised[i]) {
        const float m_new = fmaxf(m_run, mx);
        alpha[i] = fast_exp2((m_run - m_new) * c);
        m_run = m_new;
      }
      reference[i] = m_run;
    }
  };
  // Probabilities of this wavefront's blocks to LDS, as the B operand of P V.
  auto probabilities = [&](int r) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int blk = w * U + u;
      if (rows_left(2 * r + (blk >> 1)) > 32 * (blk & 1)) {
        const float mc = (blk >> 1 ? reference[1] : reference[0]) * c;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          bf16x8 pb;
#pragma unroll
          for (int i = 0; i < 8; ++i) pb[i] = static_cast<bf16_t>(fast_exp2(fmaf(s[u][8 * h + i], c, -mc)));
          *reinterpret_cast<bf16x8*>(p_set + (2 * blk + h) * 1024) = pb;
        }
      }
    }
  };
  // O^T += V^T P^T for this wavefront's 32 columns over round r's keys, and the row sums (every wavefront of the set forms
  // the same ones).  Chunks of 16 keys without a valid one have probability zero.
  auto accumulate = [&](int r) {
    const char* vt = short_lds + Lds::V + (r & (STAGES - 1)) * (2 * TILE_BYTES) + v_off[w];
    auto rescale = [&](int i) {
      if (raised[i] && (r > 0 || i > 0)) {  // nothing to rescale in front of the first tile
        l_run *= alpha[i];
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e] *= alpha[i];
      }
    };
    union VOperand {
      struct {
        s16x4 lo, hi;
      } h;
      bf16x8 v;
    };
    union POperand {
      bf16x8 v;
      bf16x2 h[4];
    };
    VOperand va[8];
    POperand pb[8];
    auto read = [&](int chunk) {
      const char* base = vt + 16 * chunk * ROW_BYTES;
      va[chunk].h.lo = lds_read_tr16(reinterpret_cast<const bf16_t*>(base));
      va[chunk].h.hi = lds_read_tr16(reinterpret_cast<const bf16_t*>(base + 8 * ROW_BYTES));
      pb[chunk].v = *reinterpret_cast<const bf16x8*>(p_set + chunk * 1024);
    };
    auto add = [&](int chunk) {
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[chunk].v, pb[chunk].v, o, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) l_run = __builtin_amdgcn_fdot2_f32_bf16(pb[chunk].h[e], ones, l_run, false);
    };
    const int left0 = rows_left(2 * r), left1 = rows_left(2 * r + 1);
#pragma unroll
    for (int chunk = 0; chunk < 4; ++chunk) read(chunk);
    if (left1 > 0) {
#pragma unroll
      for (int chunk = 4; chunk < 8; ++chunk) read(chunk);
    }
    fence();
    rescale(0);
#pragma unroll
    for (int chunk = 0; chunk < 4; ++chunk)
      if (16 * chunk < left0) add(chunk);
    rescale(1);
#pragma unroll
    for (int chunk = 0; chunk < 4; ++chunk)
      if (16 * chunk < left1) add(4 + chunk);
  };

  __syncthreads();  // (1) the query rows and K(0) are there
  {
    const char* q_rows = short_lds + Lds::P + set * (32 * ROW_BYTES);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(q_rows + k_off[ks]);
  }
  if (active) scores(0);
  for (int r = 0;; ++r) {
    __syncthreads();  // (2) the maxima of round r are there; the query rows, V(r - 1) and its probabilities have been read
    if (active) {
      follow_reference();
      probabilities(r);
    }
    __syncthreads();  // (3) V(r), K(r + 1) and the probabilities are there
    if (active) {
      accumulate(r);
      if (r + 1 < rounds) scores(r + 1);
    }
    if (r + 1 == rounds) break;
  }
  if (!active) return;

  // A lane owns 16 columns of one query row, four at a time: through LDS (2 KB per wavefront in the K tiles of the last
  // round, which all have read) into 64-byte pieces of whole rows.
  const float inv = 1.f / sum_halves(l_run);
  char* stage = short_lds + Lds::K + wave * 2048;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = static_cast<bf16_t>(o[4 * g + e] * inv);
    *reinterpret_cast<bf16x4*>(stage + n * 64 + ((g ^ ((n >> 2) & 3)) << 4) + 8 * hl) = v;
  }
  char* op = static_cast<char*>(p.out) + cur_off + static_cast<long long>(q_row0) * ROW_BYTES + w * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 16 * i + (lane >> 2), slot = lane & 3;
    const uint4 v = *reinterpret_cast<const uint4*>(stage + row * 64 + ((slot ^ ((row >> 2) & 3)) << 4));
    if (q_row0 + row < t_k) *reinterpret_cast<uint4*>(op + row * ROW_BYTES + slot * 16) = v;
  }
}

template <int D, int STAGES>
hipError_t allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_short_kernel<D, STAGES>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, ShortLds<D, STAGES>::BYTES);
}

}  // namespace

hipError_t attend_short_prepare() {
  hipError_t e = allow_lds<128, 1>();
  if (e == hipSuccess) e = allow_lds<128, 2>();
  return e;
}

// Where this kernel is the faster one.  Times of a launch in a captured graph, the other kernels -> this one.
//   One round, d = 128: 5.2 -> 3.6 us (4 to 256 pairs, 16 + 14 keys), 11.3 -> 7.8 (1024 pairs).  Beyond 32 queries it takes
//   more workgroups than the other kernel, each of which fetches the keys: 384 of them 5.9 -> 4.9 us (36 + 55 keys; with the
//   cache update 7.1 -> 6.7), 512 5.9 -> 5.1 (7.4 -> 8.2), 1024 8.2 -> 8.9.
//   One round, d = 64: 4.2 -> 3.5 us up to 256 workgroups; with the cache update 4.6 -> 3.9, for 512 of them 5.4 -> 6.1.
//   More rounds, d = 128: two stages leave room for one workgroup per compute unit.  Up to 256 of them 7.2 -> 5.4 us (64 + 140
//   keys), 13.2 -> 10.0 (144 + 385), 20.5 -> 17.6 (324 + 807); 25.2 -> 24.2 for 27 tiles, 33.3 -> 34.1 for 40.  288
//   take a second turn: 9.4 -> 12.4.  The workgroups of the cache update take as much room and wait for a unit; how many of them
//   the walks hide depends on their length (inputs in cache; inputs from memory).  256 + 160 of 9 tiles 14.4 -> 14.5; 16.4 -> 16.8,
//   240 + 111 of 5 tiles 10.6 -> 10.8; 11.9 -> 12.4, 256 + 192 of 5 tiles 11.6 -> 12.3; 13.9 -> 14.1; but 192 + 160 of 8 tiles
//   13.4 -> 11.3; 15.1 -> 13.4, 224 + 160 of 10 tiles 15.5 -> 13.4; 17.3 -> 16.1, 256 + 170 of 13 tiles 19.6 -> 19.1; 23.6 -> 21.0.
//   More rounds, d = 64: 0.94 to 1.09 times the other kernel's time.
// Never for queries off the 4-byte grid: they come by the copies into LDS here, in the other kernels by ordinary loads.
// Never where two key streams may be taken (attend.hip): their outputs have other last bits, and whether a launch carries
// the cache update must not show in its outputs.
bool attend_short_fits(const AttendParams& p, int d, int max_len, unsigned copy_blocks) {
  if (reinterpret_cast<unsigned long long>(p.q) % 4 != 0) return false;
  const int tiles = (p.t_k + tile::ROWS - 1) / tile::ROWS + (max_len + tile::ROWS - 1) / tile::ROWS;
  const int queries = 32 * (128 / d);  // per workgroup
  const unsigned pairs8 = (unsigned(p.H) * p.batch + 7) / 8 * 8;
  const unsigned long long blocks = (unsigned long long)((p.t_k + queries - 1) / queries) * pairs8;
  if (tiles <= 2 && d == 64) return blocks <= 256;
  if (tiles <= 2) return p.t_k <= queries || blocks <= (copy_blocks ? 384 : 512);
  return d == 128 && p.t_k < TWO_STREAM_MIN_TOKENS && tiles <= 24 && blocks <= 256 &&
         blocks + copy_blocks <= unsigned(std::min(272 + 12 * tiles, 480));
}

hipError_t launch_attend_short(AttendParams p, int d, int max_len, unsigned copy_blocks, hipStream_t stream) {
  const int queries = 32 * (128 / d);
  p.n_qtiles = (p.t_k + queries - 1) / queries;
  const unsigned pairs8 = (unsigned(p.H) * p.batch + 7) / 8 * 8;  // padded so that id % 8 is the XCD
  p.attend_blocks = int(unsigned(p.n_qtiles) * pairs8);
  p.div_qtiles = reciprocal(p.attend_blocks, p.n_qtiles);
  p.div_batch = reciprocal(pairs8, p.batch);
  const dim3 grid(unsigned(p.attend_blocks) + copy_blocks), block(512);
  if (d == 64)
    hipLaunchKernelGGL((attend_short_kernel<64, 1>), grid, block, (ShortLds<64, 1>::BYTES), stream, p);
  else if ((p.t_k + tile::ROWS - 1) / tile::ROWS + (max_len + tile::ROWS - 1) / tile::ROWS <= 2)
    hipLaunchKernelGGL((attend_short_kernel<128, 1>), grid, block, (ShortLds<128, 1>::BYTES), stream, p);
  else
    hipLaunchKernelGGL((attend_short_kernel<128, 2>), grid, block, (ShortLds<128, 2>::BYTES), stream, p);
  return hipGetLastError();
}

}  // namespace heatkv
