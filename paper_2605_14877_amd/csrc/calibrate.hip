// Scale attention mass (Sec. 3.1, Eq. 2): for the queries of scale k1 over the
// uncompressed keys of scales 0..k1, the softmax mass that falls inside each
// key block k2, averaged over the query rows.
//
// The attention matrix is never materialised.  Key tiles never straddle two
// scale blocks; per query row the kernel keeps one running maximum and, for the
// block being walked, a sum of exponentials relative to that maximum.  At the
// end of a block the pair (sum, maximum at that moment) is parked in LDS; after
// the last block every parked sum is rescaled to the final maximum, which gives
// the row's normaliser and its per-block masses at once.  Row masses are then
// summed over 128 rows at a time in a fixed order and written as one partial per
// (head, 128 query rows); a second kernel adds the partials in row order, so the
// result is bit-reproducible (no floating-point atomics anywhere).
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "device_util.h"
#include "f32_mfma.h"
#include "f32_split.h"
#include "kernels.h"
#include "launch_rules.h"
#include "tile_lds.h"

namespace heatkv {

namespace {

constexpr int MAXK = HEATKV_MAX_SCALES;

// One query scale of a launch.  A launch may cover several (calibration data of all scales is available at
// once, unlike generation); their workgroups are laid out one scale after the other, largest scale first.
struct ScaleJob {
  int k1;
  int block_begin;  // first workgroup id of this scale (a multiple of 8)
  const void *q, *k_all;
  float* partial;  // [batch*H][n_qtiles][K]
};

struct CalibParams {
  int H, batch, K, n_scales;
  int t[MAXK];
  int c[MAXK];  // c[k] = t[0] + .. + t[k]
  ScaleJob job[MAXK];
  float sm_scale;
};

// Where the masses of a launch of one query tile go, and the table that they are added to.
struct CalibDirect {
  float *mass, *beta;  // mass may be null
  float weight;
  int layer;
};

// The kernel arguments take more than a kilobyte, and which of them a workgroup needs follows from others: read one
// after the other they are a chain of scalar-cache misses.  This asks for their lines together.
__device__ __forceinline__ void touch_params(const CalibParams& p) {
  asm volatile("; kernel arguments" ::"s"(p.n_scales), "s"(p.t[13]), "s"(p.t[29]), "s"(p.c[14]), "s"(p.job[0].k1),
               "s"(p.job[1].block_begin), "s"(p.sm_scale));
}

// The scale a workgroup belongs to (workgroup-uniform, a handful of scalar compares).
__device__ __forceinline__ int scale_of_block(const CalibParams& p, int block) {
  int si = 0;
  while (si + 1 < p.n_scales && block >= p.job[si + 1].block_begin) ++si;
  return si;
}

// ---------------------------------------------------------------------------
// bf16, d = 128 or 64: S^T = K Q^T on the matrix cores, one lane per query column
// (same operand layout, LDS tile format and HBM -> LDS copy as the attention
// kernel).  Two instances.  CSETS = 1: 128 queries per workgroup, one set of 32 per
// wavefront, three workgroups per compute unit.  CSETS = 2: 256 queries per
// workgroup; every wavefront owns two sets of 32 (rows w*32 + n and 128 + w*32 + n
// of the tile) and runs both against each K operand it has read from LDS, so a K
// tile is copied and read once per 256 queries and the matrix-core work of one set
// overlaps the exponentials of the other inside the wavefront; two workgroups per
// compute unit.  The launcher takes the second when its workgroups fill their 512
// slots at least once.
// ---------------------------------------------------------------------------
constexpr int CBM1 = 128;  // queries per set of four wavefronts
constexpr int CBN = tile::ROWS;

// Dynamic LDS: two K tiles, then blk_sum[k1+1][rows], blk_max[k1+1][rows], fin_max[rows] (floats), rows = the
// queries of a workgroup.
__host__ __device__ constexpr size_t calib_lds_bytes(int k1, int csets, int d) {
  return 2 * size_t(CBN * 2 * d) + (2 * size_t(k1 + 1) + 1) * (CBM1 * csets) * sizeof(float);
}

template <int CSETS, int CD>
__global__ __launch_bounds__(256, CSETS == 1 ? 3 : 2) void calibrate_bf16_kernel(CalibParams p) {
  static_assert(CD == 128 || CD == 64, "head dimension 128 or 64");
  constexpr int CROW_BYTES = 2 * CD;            // one bf16 row
  constexpr int CTILE_BYTES = CBN * CROW_BYTES;  // 16 KB or 8 KB
  constexpr int NK = CD / 16;                    // MFMA steps of a score block
  constexpr int CBM = CBM1 * CSETS;  // queries per workgroup
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const ScaleJob& job = p.job[scale_of_block(p, blockIdx.x)];
  const int k1 = job.k1, t_k1 = p.t[k1];
  const int n_qtiles = (t_k1 + CBM - 1) / CBM;
  const int block = blockIdx.x - job.block_begin;
  float* blk_sum = reinterpret_cast<float*>(lds + 2 * CTILE_BYTES);
  float* blk_max = blk_sum + (k1 + 1) * CBM;
  float* fin_max = blk_max + (k1 + 1) * CBM;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hl = lane >> 5;

  // All query tiles of one (batch row, head) read the same keys: give them ids on one XCD (id % 8).
  const int xcd = block & 7, slot = block >> 3;  // block_begin is a multiple of 8: block & 7 is the hardware XCD
  const int bh = (slot / n_qtiles) * 8 + xcd;
  if (bh >= p.batch * p.H) return;
  const int qt = slot % n_qtiles;
  const int c_k1 = p.c[k1];

  const char* kbase = reinterpret_cast<const char*>(static_cast<const bf16_t*>(job.k_all) +
                                                    static_cast<long long>(bh) * c_k1 * CD);
  // The second set of a tile exists only if the tile reaches past its first 128 rows (workgroup-uniform).
  const bool two_sets = CSETS == 2 && qt * CBM + 128 < t_k1;
  bf16x8 qreg[CSETS][NK];
#pragma unroll
  for (int qs = 0; qs < CSETS; ++qs) {
    const int q_row = qt * CBM + qs * 128 + wave * 32 + n;
    const int ld = q_row < t_k1 ? q_row : t_k1 - 1;
    const bf16_t* qp = static_cast<const bf16_t*>(job.q) + (static_cast<long long>(bh) * t_k1 + ld) * CD + 8 * hl;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) qreg[qs][ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
  }
  const float c = p.sm_scale * kLog2e;

  // HBM -> LDS copy of one K tile in the tile format shared with the attention kernel (tile_lds.h: raw
  // global_load_lds, explicit ordering by s_waitcnt vmcnt + barrier).
  const int ld_off = tile::loader_off_k<CROW_BYTES>(wave, lane);
  const unsigned lds_base =
      static_cast<unsigned>(reinterpret_cast<unsigned long long>((__attribute__((address_space(3))) char*)(&lds[0])));
  auto issue_tile = [&](int k2, int tile_i, int buf) {
    const int left = p.t[k2] - tile_i * CBN;
    const char* kb = kbase + static_cast<long long>(p.c[k2] - p.t[k2] + tile_i * CBN) * CROW_BYTES;
    const unsigned kd = lds_base + buf * CTILE_BYTES;
    if (left >= CBN)
      tile::issue_full<CROW_BYTES>(kd, wave, ld_off, kb);
    else  // ragged tile: rows past the end re-read the last valid row
      tile::issue_ragged<false, CROW_BYTES>(kd, wave, lane, left, kb);
  };
  int k_off[NK];
  tile::reader_off_k<CROW_BYTES>(lane, k_off);

  float m_run[CSETS], cur[CSETS];
#pragma unroll
  for (int qs = 0; qs < CSETS; ++qs) {
    m_run[qs] = lowest_reference(c);
    cur[qs] = 0.f;
  }
  int k2 = 0, tile = 0;  // the tile being computed

  // Adds a tile's probabilities (rs: four partial sums of this lane's 32, relative to m_run) to the block's sum.
  // Probabilities are taken relative to the running reference m_run, which is only brought up to the true
  // row maximum when it has fallen too far behind: as long as no score exceeds it by more than 8 in the
  // base-2 exponent a lane's 32 probabilities of the tile sum to at most 2^13, so a larger sum or an
  // infinity (the first tile, where m_run still is the lowest reference) sends the whole wavefront through the
  // exact path, which finds the tile maximum, rescales what the block has summed so far and redoes the tile's
  // exponentials.  The masses are ratios of such sums, so they do not depend on the reference; the max
  // chain, one vector instruction per two scores, leaves the common path.
  auto fold = [&](int qs, const f32x16 (&s)[2], float (&rs)[4], int block, bool last_of_block) {
    float tile_sum = (rs[0] + rs[1]) + (rs[2] + rs[3]);
    if (__any(!(tile_sum <= 8192.f))) {
      float mx = s[0][0];
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[cb][r]);
      mx = max_halves(mx);
      const float m_new = fmaxf(m_run[qs], mx);
      cur[qs] *= fast_exp2((m_run[qs] - m_new) * c);
      m_run[qs] = m_new;
      const float mc = m_new * c;
#pragma unroll
      for (int i = 0; i < 4; ++i) rs[i] = 0.f;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) rs[r & 3] += fast_exp2(fmaf(s[cb][r], c, -mc));
      tile_sum = (rs[0] + rs[1]) + (rs[2] + rs[3]);
    }
    cur[qs] += tile_sum;
    if (last_of_block) {
      const float both = sum_halves(cur[qs]);
      if (hl == 0) {
        blk_sum[block * CBM + qs * 128 + wave * 32 + n] = both;
        blk_max[block * CBM + qs * 128 + wave * 32 + n] = m_run[qs];
      }
      cur[qs] = 0.f;
    }
  };

  // A step of the one-set instance, in the compiler's order.
  auto tile_step = [&](auto buf_tag) {
    constexpr int buf = decltype(buf_tag)::value;
    // successor of (k2, tile) in block-major order
    const int tiles_here = (p.t[k2] + CBN - 1) / CBN;
    const bool last_of_block = tile + 1 >= tiles_here;
    const int nk2 = last_of_block ? k2 + 1 : k2, ntile = last_of_block ? 0 : tile + 1;
    wait_vmcnt<0>();
    __syncthreads();
    if (nk2 <= k1) issue_tile(nk2, ntile, buf ^ 1);
    const char* kt = lds + buf * CTILE_BYTES;

    bf16x8 ka[2][NK];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        ka[cb][ks] = *reinterpret_cast<const bf16x8*>(kt + cb * 32 * CROW_BYTES + k_off[ks]);
    const int left = p.t[k2] - tile * CBN;
    f32x16 s[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[cb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        s[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[cb][ks], qreg[0][ks], s[cb], 0, 0, 0);
    // all sixteen operand reads go out before the first MFMA instead of two at a time
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * NK, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * NK, 0);
    if (left < CBN) tile::mask_rows(left, hl, s);
    const float mc = m_run[0] * c;
    float rs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) rs[r & 3] += fast_exp2(fmaf(s[cb][r], c, -mc));
    fold(0, s, rs, k2, last_of_block);
    k2 = nk2;
    tile = ntile;
  };

  // The walk of the two-set instance, issue order fixed by hand.  Per tile two phases of 2 NK slots, one MFMA each:
  //   A: scores of set 0; in its slots the exponentials of set 1 of the tile before
  //   B: scores of set 1; in its slots the exponentials of set 0, the K operands of the next tile (each into the
  //      registers that its MFMA has just read) and the copies of the tile after that
  // The barrier stands between A and B: by then every wavefront has this tile's operands in registers, so its stage is
  // free for the copies, and the next tile, copied during the phase B before, has landed.  No operand read stands
  // between a barrier and the MFMAs that need it.
  // Bound: the vector ALU (three instructions per score, busy 77 % of the time that wavefronts are resident) next to the
  // matrix pipes (62 %), at the 1.85 GHz that this mix leaves.  All 13 scales of a 2B-like layer (16 heads, batch 2): 558
  // -> 531 us, 1.06 PFLOP/s.  Exponent, exponential and sum of a probability in three successive slots: no faster.
  auto two_set_walk = [&](auto two_tag) {
    constexpr bool kTwo = decltype(two_tag)::value;  // a last tile of at most 128 rows has no set 1
    struct Tile {
      int k2, left;  // block, rows from the tile's first one to the block's end; left = 0: past the walk's end
    };
    const char* kb = kbase;  // first row of the tile that is fetched next
    Tile next{0, p.t[0]};    // that tile
    auto advance = [&] {     // sizes of blocks are read only when the walk enters one
      if (next.left > CBN) {
        kb += CTILE_BYTES;
        next.left -= CBN;
      } else {
        kb += static_cast<long long>(next.left) * CROW_BYTES;
        ++next.k2;
        next.left = next.k2 <= k1 ? p.t[next.k2] : 0;
      }
    };
    constexpr int CPT = CTILE_BYTES / 4096;  // copies of a tile per wavefront
    auto copy = [&](const tile::Descriptor& src, int buf, int i) {
      tile::copy_1k_checked(lds_base + wave * 1024, buf * CTILE_BYTES + i * 4096, ld_off, src, i * 4096);
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
    auto mask_tail = [&](int left, f32x16 (&s)[2]) {
      if (left < CBN) tile::mask_rows(left, hl, s);
    };
    auto load_k = [&](bf16x8& dst, int buf, int cb, int ks) {
      dst = *reinterpret_cast<const bf16x8*>(lds + buf * CTILE_BYTES + cb * 32 * CROW_BYTES + k_off[ks]);
    };
    bf16x8 ka[2][NK];
    f32x16 s[2][2];  // [set][block of 32 keys]
    float rs[4];
    // Slot i's share of set qs's probabilities, summed in the order of the exact path.
    constexpr int PER_SLOT = 16 / NK;
    auto exps = [&](int qs, float mc, int i) {
#pragma unroll
      for (int u = 0; u < PER_SLOT; ++u) {
        const int r = i * PER_SLOT + u;
        rs[r & 3] += fast_exp2(fmaf(s[qs][r >> 4][r & 15], c, -mc));
      }
    };
    auto settle = [&](int qs, const Tile& t) { fold(qs, s[qs], rs, t.k2, t.left <= CBN); };

    Tile now = next;
    const tile::Descriptor d0 = tile::tile_descriptor<CROW_BYTES>(kb, next.left);
    advance();
    const tile::Descriptor d1 = tile::tile_descriptor<CROW_BYTES>(kb, next.left);
    Tile ahead = next;
    advance();
#pragma unroll
    for (int i = 0; i < CPT; ++i) copy(d0, 0, i);
#pragma unroll
    for (int i = 0; i < CPT; ++i) copy(d1, 1, i);
    wait_vmcnt<CPT>();
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) load_k(ka[cb][ks], 0, cb, ks);
    Tile before{0, 0};  // the tile whose set 1 is still to be summed
    auto step = [&](auto buf_tag, auto first_tag) {
      constexpr int buf = decltype(buf_tag)::value;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[0][cb][r] = 0.f;
      const float mc1 = m_run[1] * c;
#pragma unroll
      for (int i = 0; i < 4; ++i) rs[i] = 0.f;
      fence();
      if constexpr (kTwo && !decltype(first_tag)::value) {
#pragma unroll
        for (int i = 0; i < 2 * NK; ++i) {
          s[0][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i & 1][i >> 1], qreg[0][i >> 1], s[0][i & 1], 0, 0, 0);
          fence();
          exps(1, mc1, i);
          fence();
        }
        settle(1, before);
      } else {
#pragma unroll
        for (int i = 0; i < 2 * NK; ++i)
          s[0][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i & 1][i >> 1], qreg[0][i >> 1], s[0][i & 1], 0, 0, 0);
      }
      const tile::Descriptor src = tile::tile_descriptor<CROW_BYTES>(kb, next.left);
      wait_vmcnt<0>();
      __syncthreads();
      mask_tail(now.left, s[0]);
      const float mc0 = m_run[0] * c;
#pragma unroll
      for (int i = 0; i < 4; ++i) rs[i] = 0.f;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[1][cb][r] = 0.f;
      fence();
      if constexpr (kTwo) {
#pragma unroll
        for (int i = 0; i < 2 * NK; ++i) {
          s[1][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i & 1][i >> 1], qreg[1][i >> 1], s[1][i & 1], 0, 0, 0);
          fence();
          load_k(ka[i & 1][i >> 1], buf ^ 1, i & 1, i >> 1);
          if (i < CPT) copy(src, buf, i);
          exps(0, mc0, i);
          fence();
        }
        settle(0, now);
        mask_tail(now.left, s[1]);
      } else {
#pragma unroll
        for (int i = 0; i < 2 * NK; ++i) {
          load_k(ka[i & 1][i >> 1], buf ^ 1, i & 1, i >> 1);
          if (i < CPT) copy(src, buf, i);
          exps(0, mc0, i);
        }
        settle(0, now);
      }
      before = now;
      now = ahead;
      ahead = next;
      advance();
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    step(Even{}, std::true_type{});
    while (now.left > 0) {
      step(Odd{}, std::false_type{});
      if (now.left == 0) break;
      step(Even{}, std::false_type{});
    }
    if constexpr (kTwo) {
      const float mc1 = m_run[1] * c;
#pragma unroll
      for (int i = 0; i < 4; ++i) rs[i] = 0.f;
#pragma unroll
      for (int i = 0; i < 2 * NK; ++i) exps(1, mc1, i);
      settle(1, before);
    }
    wait_vmcnt<0>();  // the copies past the end (no rows: zeros) land before the workgroup ends
  };

  if constexpr (CSETS == 2) {
    if (two_sets)
      two_set_walk(std::true_type{});
    else
      two_set_walk(std::false_type{});
  } else {
    issue_tile(0, 0, 0);
    while (true) {
      tile_step(std::integral_constant<int, 0>{});
      if (k2 > k1) break;
      tile_step(std::integral_constant<int, 1>{});
      if (k2 > k1) break;
    }
  }
  if (hl == 0) {
#pragma unroll
    for (int qs = 0; qs < CSETS; ++qs) fin_max[qs * 128 + wave * 32 + n] = m_run[qs];
  }
  __syncthreads();

  // Row masses relative to the final maximum, normalised; rows past t_k1 contribute nothing.
  if (tid < 128 || two_sets) {  // one thread per query row of the tile; rows of an absent second set hold nothing
    const float mf = fin_max[tid];
    float l = 0.f;
    for (int j = 0; j <= k1; ++j) {
      const float w = blk_sum[j * CBM + tid] * fast_exp2((blk_max[j * CBM + tid] - mf) * c);
      blk_sum[j * CBM + tid] = w;
      l += w;
    }
    const float inv = (qt * CBM + tid < t_k1) ? 1.f / l : 0.f;
    for (int j = 0; j <= k1; ++j) blk_sum[j * CBM + tid] *= inv;
  }
  __syncthreads();
  // One partial per 128 query rows whichever the instance: a set of the two-set instance holds exactly the rows of
  // one query tile of the other and sums them in the same order, so both write the same bits to the same places.
  const int n_parts = (t_k1 + CBM1 - 1) / CBM1;
  for (int j = wave; j <= k1; j += 4) {
#pragma unroll
    for (int qs = 0; qs < CSETS; ++qs) {
      if (qs == 1 && !two_sets) break;
      float v = blk_sum[j * CBM + qs * CBM1 + lane] + blk_sum[j * CBM + qs * CBM1 + lane + 64];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
      if (lane == 0) job.partial[(static_cast<long long>(bh) * n_parts + CSETS * qt + qs) * p.K + j] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// fp32: S^T = K Q^T on the fp32 matrix instructions (f32_mfma.h), 16 queries per workgroup.  The key tiles (16 rows,
// block-major) are dealt round robin to the four wavefronts; a lane keeps the running maximum and the sum of the
// block being walked for its own keys, the lane groups are combined when the wavefront leaves a block and the
// wavefronts at the end, all in a fixed order.
//
// Bound: start-up below about 100 query rows (4.4 us of kernel for one tile), the matrix pipe with the step's vector
// instructions and one or two workgroups per compute unit above (16 heads, 400 x 937, d = 128: 27.5 us = 56 TFLOP/s;
// the vector-ALU kernel that this one replaced: 261 us).  Keys straight into registers instead of through the stage:
// 34 us; sizes of blocks looked up in every step: 33 us; kernel arguments read one after the other: +0.8 us per launch.
// ---------------------------------------------------------------------------
constexpr int FQ = f32m::TILE;
constexpr int FW = 4;           // wavefronts that share a query tile

// Dynamic LDS of a query tile: key stages [FW], final maxima [FW][FQ] and inverse row sums [FQ], then block sums and references
// [k1+1][2][FW][FQ], rounded up to whole kilobytes.
template <int D>
__host__ __device__ constexpr size_t f32_lds_bytes(int k1) {
  const size_t b = FW * f32m::KeyStage<D>::BYTES + ((2 * size_t(k1 + 1) + 1) * FW + 1) * FQ * sizeof(float);
  return (b + 1023) / 1024 * 1024;
}

// G > 0: one query scale of at most FQ rows, G batch rows.  A workgroup takes a head, G times four wavefronts its batch rows,
// and the row masses of the one query tile are all there is to average: the workgroup divides them by the number of rows and
// adds them up as the reduction below does, bit for bit, and there is no second launch.  In a captured graph: 8 heads, batch 2,
// d = 128, 1 x 1 and 16 x 21 keys 5.7 -> 4.7 and 6.3 -> 5.8 us; 4 heads, batch 1, d = 64, 1 x 1 and 16 x 21 5.0 -> 3.5 and 5.4 -> 3.8.
template <int D, int G>
__global__ __launch_bounds__(64 * FW * (G > 0 ? G : 1)) void calibrate_f32_kernel(CalibParams p, CalibDirect direct) {
  using Stage = f32m::KeyStage<D>;
  extern __shared__ __attribute__((aligned(1024))) char calib_f32_lds[];

  const int group = G > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * FW)) : 0;
  const int tid = G > 1 ? threadIdx.x % (64 * FW) : threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_params(p);
  const ScaleJob& job = p.job[scale_of_block(p, blockIdx.x)];
  const int k1 = job.k1, t_k1 = p.t[k1];
  const int n_qtiles = (t_k1 + FQ - 1) / FQ;
  const int block = blockIdx.x - job.block_begin;
  const int xcd = block & 7, slot = block >> 3;  // all query tiles of a (batch row, head) on one XCD
  const int bh = G > 0 ? group * p.H + block : (slot / n_qtiles) * 8 + xcd;
  if (bh >= p.batch * p.H) return;
  const int qt = G > 0 ? 0 : slot % n_qtiles;
  const int q_rows = min(t_k1 - qt * FQ, FQ);
  const float* kbase = static_cast<const float*>(job.k_all) + static_cast<long long>(bh) * p.c[k1] * D;

  char* const lds = calib_f32_lds + group * f32_lds_bytes<D>(k1);
  float(*const fin_max)[FQ] = reinterpret_cast<float(*)[FQ]>(lds + FW * Stage::BYTES);
  float* const row_inv = fin_max[FW];
  constexpr int BLOCKS = FW * Stage::BYTES + (FW + 1) * FQ * 4;
  float(*const blk)[2][FW][FQ] = reinterpret_cast<float(*)[2][FW][FQ]>(lds + BLOCKS);  // [.][0] sums, [.][1] references
  char* const stage = lds + wave * Stage::BYTES;
  const Stage keys(stage, lane);
  f32m::Rows<D> q, k;
  q.load(static_cast<const float*>(job.q) + (static_cast<long long>(bh) * t_k1 + qt * FQ) * D, q_rows, lane);

  // The wavefront's tile: number `tile` of block k2, which has rows_left rows from that tile on.  `first` is the tile's
  // first key.  Sizes of blocks are read only when the walk enters one: a step that stays inside its block reads no
  // tables.
  int k2 = 0, first = 0, rows_left = 0;
  auto enter = [&](int tile) {  // tile number counted from the start of block k2; carries it over to the block that has it
    while (k2 <= k1) {
      const int rows = p.t[k2], here = (rows + FQ - 1) / FQ;
      if (tile < here) {
        first = p.c[k2] - rows + tile * FQ;
        rows_left = rows - tile * FQ;
        return;
      }
      tile -= here;
      ++k2;
    }
  };
  auto fetch = [&] { keys.fill(kbase + static_cast<long long>(first) * D, min(rows_left, FQ), lane); };
  for (int j = 0; j <= k1; ++j)  // blocks without a tile of this wavefront
    if (g == 0) {
      blk[j][0][wave][n] = 0.f;
      blk[j][1][wave][n] = f32m::LOWEST;
    }
  enter(wave);
  if (k2 <= k1) fetch();
  const f32m::Exponent prob(p.sm_scale);
  float m = f32m::LOWEST, cur = 0.f;
  while (k2 <= k1) {
    const int here = k2, rows = rows_left;
    Stage::take(k, stage, lane);
    if (rows_left > FW * FQ) {
      first += FW * FQ;
      rows_left -= FW * FQ;
    } else {
      const int tiles_left = (rows_left + FQ - 1) / FQ;  // of this block, from the tile on: at most FW
      ++k2;
      enter(FW - tiles_left);
    }
    if (k2 <= k1) fetch();
    f32x4 s = f32m::scores<D>(k, q);
    s *= prob.c;
    if (rows < FQ) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * g + r >= rows) s[r] = -INFINITY;
    }
    const float m_new = fmaxf(m, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
    cur *= prob(m, m_new);
    m = m_new;
    cur += (prob(s[0], m) + prob(s[1], m)) + (prob(s[2], m) + prob(s[3], m));
    if (k2 != here) {  // the wavefront leaves the block
      const float mb = f32m::max_groups(m);
      const float sb = f32m::sum_groups_product(cur, prob(m, mb));
      if (g == 0) {
        blk[here][0][wave][n] = sb;
        blk[here][1][wave][n] = mb;
      }
      cur = 0.f;
    }
  }
  m = f32m::max_groups(m);
  if (g == 0) fin_max[wave][n] = m;
  __syncthreads();

  // Row masses relative to the final maximum, normalised; rows past t_k1 contribute nothing.
  {
    const int row = tid & (FQ - 1);
    float mf = fin_max[0][row];
#pragma unroll
    for (int w = 1; w < FW; ++w) mf = fmaxf(mf, fin_max[w][row]);
    for (int j = tid / FQ; j <= k1; j += 64 * FW / FQ) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < FW; ++w) v += blk[j][0][w][row] * prob(blk[j][1][w][row], mf);
      blk[j][0][0][row] = v;
    }
  }
  __syncthreads();
  if (tid < FQ) {
    float l = 0.f;
    for (int j = 0; j <= k1; ++j) l += blk[j][0][0][tid];
    row_inv[tid] = tid < q_rows ? 1.f / l : 0.f;
  }
  __syncthreads();
  if (tid <= k1) {
    float v = 0.f;
#pragma unroll
    for (int rr = 0; rr < FQ; ++rr) v += blk[tid][0][0][rr] * row_inv[rr];
    if constexpr (G > 0)
      blk[tid][0][1][0] = v / static_cast<float>(t_k1);
    else
      job.partial[(static_cast<long long>(bh) * n_qtiles + qt) * p.K + tid] = v;
  }
  if constexpr (G > 0) {
    __syncthreads();
    const int j = tid;
    if (j >= p.K) return;
    if (direct.mass) direct.mass[static_cast<long long>(bh) * p.K + j] = j <= k1 ? blk[j][0][1][0] : 0.f;
    if (group > 0) return;
    float acc = 0.f;
    for (int b = 0; b < G; ++b) {
      const auto* sums = reinterpret_cast<const float(*)[2][FW][FQ]>(calib_f32_lds + b * f32_lds_bytes<D>(k1) + BLOCKS);
      acc += j <= k1 ? sums[j][0][1][0] : 0.f;
    }
    float* const out = direct.beta + ((static_cast<long long>(direct.layer) * p.H + block) * p.K + k1) * p.K + j;
    *out = *out + direct.weight * acc;
  }
}

// ---------------------------------------------------------------------------
// fp32 scales of many query rows: S^T = K Q^T on the bf16 matrix instructions, operands in three bf16 parts (f32_split.h).
// 32 queries per workgroup, whose parts every wavefront keeps in registers; key tiles of 32 rows dealt round robin to
// eight wavefronts.  Otherwise as above.  Error of the masses against 64 bits on the same inputs (16 kinds, 40 seeds each): 1.002
// +- 0.005 times that of the kernel above, 7e-8 to 1.1e-7.  Bound: vector instructions, 48 for the six products of a step, as in
// the attention kernel (attend_f32_split.hip).  d = 128: 256 pairs, 625 x 2511 keys 976 -> 834 us.
// ---------------------------------------------------------------------------
constexpr int SQ = 32;  // queries of a workgroup, keys of a tile
constexpr int SW = 8;   // wavefronts
constexpr int kMaxLds = 160 * 1024;

template <int D>
struct SplitLds {
  static constexpr int ROW = 4 * D, STAGE = SQ * ROW;
  static constexpr int BLOCKS = SW * STAGE;            // block sums and references; at first the parts of the query rows
  static constexpr int PARTS = 3 * (D / 16) * 1024;
  static constexpr int PER_BLOCK = 2 * SW * SQ * 4;    // [sum, maximum][wavefront][query]
  static constexpr int REST = SW * SQ * 4 + SQ * 4 + SW * 4;  // final maxima, inverse row sums, flags
  __host__ __device__ static constexpr size_t bytes(int k1) {
    return BLOCKS + (PARTS > (k1 + 1) * PER_BLOCK ? PARTS : (k1 + 1) * PER_BLOCK) + REST;
  }
};

template <int D>
__global__ __launch_bounds__(64 * SW) void calibrate_f32_split_kernel(CalibParams p) {
  using Lds = SplitLds<D>;
  constexpr int NK = D / 16, ROW = Lds::ROW, CPR = D / 4;
  constexpr int COPIES = Lds::STAGE / 1024, ROWS = 64 / CPR;  // copies of a tile, rows of one
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  touch_params(p);
  const ScaleJob& job = p.job[scale_of_block(p, blockIdx.x)];
  const int k1 = job.k1, t_k1 = p.t[k1];
  const int n_qtiles = (t_k1 + SQ - 1) / SQ;
  const int block = blockIdx.x - job.block_begin;
  const int xcd = block & 7, slot = block >> 3;  // all query tiles of a (batch row, head) on one XCD
  const int bh = (slot / n_qtiles) * 8 + xcd;
  if (bh >= p.batch * p.H) return;
  const int qt = slot % n_qtiles;
  const int q_rows = min(t_k1 - qt * SQ, SQ);
  const float* kbase = static_cast<const float*>(job.k_all) + static_cast<long long>(bh) * p.c[k1] * D;
  const int at_rest = Lds::BLOCKS + (Lds::PARTS > (k1 + 1) * Lds::PER_BLOCK ? Lds::PARTS : (k1 + 1) * Lds::PER_BLOCK);
  float* const blk = reinterpret_cast<float*>(lds + Lds::BLOCKS);
  auto blk_sum = [&](int j, int w, int row) -> float& { return blk[(2 * j * SW + w) * SQ + row]; };
  auto blk_max = [&](int j, int w, int row) -> float& { return blk[((2 * j + 1) * SW + w) * SQ + row]; };
  float* const fin_max = reinterpret_cast<float*>(lds + at_rest);
  float* const row_inv = fin_max + SW * SQ;
  int* const big = reinterpret_cast<int*>(row_inv + SQ);

  // The wavefront's tile: first row, rows from it to the end of its block k2.
  int k2 = 0, first = 0, rows_left = 0;
  auto enter = [&](int tile) {  // tile number counted from the start of block k2; carries it over to the block that has it
    while (k2 <= k1) {
      const int rows = p.t[k2], here = (rows + SQ - 1) / SQ;
      if (tile < here) {
        first = p.c[k2] - rows + tile * SQ;
        rows_left = rows - tile * SQ;
        return;
      }
      tile -= here;
      ++k2;
    }
  };
  // Rows past the tile's end are zeros; the 16-byte chunks of a row are XORed with the row number.
  const unsigned stage = static_cast<unsigned>(
      reinterpret_cast<unsigned long long>((__attribute__((address_space(3))) char*)(&lds[0]))) + wave * Lds::STAGE;
  auto fetch = [&] {
    const tile::Descriptor src =
        tile::tile_descriptor<ROW>(reinterpret_cast<const char*>(kbase + static_cast<long long>(first) * D), rows_left);
    const int b = lane / CPR;
    const int off = b * ROW + (((lane & (CPR - 1)) ^ b) << 4);  // row ROWS i + b, chunk c ^ row = (c ^ b) ^ ROWS i
#pragma unroll
    for (int i = 0; i < COPIES; ++i) tile::copy_1k_checked(stage, i * 1024, off ^ ((ROWS * i & 15) << 4), src, i * 1024);
  };
  enter(wave);
  if (k2 <= k1) fetch();

  // Query rows: wavefront `step` splits the elements 16 step + 8 hl .. + 7 of row n, all take the parts of all.
  const float* const q_row = static_cast<const float*>(job.q) +
                             (static_cast<long long>(bh) * t_k1 + qt * SQ + min(n, q_rows - 1)) * D + 8 * hl;
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
      *reinterpret_cast<bf16x8*>(lds + Lds::BLOCKS + (i * NK + wave) * 1024 + lane * 16) = parts.part(i);
  }
  const bool mine_big = __any(q_most > f32s::LARGEST);
  if (lane == 0) big[wave] = mine_big;
  __syncthreads();
  f32s::Parts qp[NK];
#pragma unroll
  for (int step = 0; step < NK; ++step)
#pragma unroll
    for (int i = 0; i < 3; ++i)
      qp[step].set(i, *reinterpret_cast<const bf16x8*>(lds + Lds::BLOCKS + (i * NK + step) * 1024 + lane * 16));
  int q_big = 0;
#pragma unroll
  for (int w = 0; w < SW; ++w) q_big |= big[w];
  q_big = __builtin_amdgcn_readfirstlane(q_big);
  __syncthreads();  // the parts' place is free
  for (int j = 0; j <= k1; ++j)  // blocks without a tile of this wavefront
    if (hl == 0) {
      blk_sum(j, wave, n) = 0.f;
      blk_max(j, wave, n) = f32m::LOWEST;
    }
  const f32m::Exponent prob(p.sm_scale);
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  float m = f32m::LOWEST, cur = 0.f;
  while (k2 <= k1) {
    const int here = k2, rows = rows_left;
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    // Chunks 4 step + 2 hl and the next one of row n, XORed with the row: address bits in which the row's own has no ones.
    unsigned k_at = stage + n * ROW + (((2 * hl) ^ (n & 15)) << 4);
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
    // Between the products of a step: the split of the next one's keys, the keys after that.
    float x[2][8], k_most = 0.f;
    f32s::Parts kp[2];
    load_k(0, x[0]);
    load_k(1, x[1]);
    k_most = f32s::magnitude(k_most, x[0]);
    f32s::split(kp[0], x[0]);
#pragma unroll
    for (int step = 0; step < NK; ++step)
#pragma unroll
      for (int i = 0; i < f32s::PRODUCTS; ++i) {
        fence();
        f32s::add_product(i, small, s, kp[step & 1], qp[step]);
        fence();
        if (i == 0 && step + 2 < NK) load_k(step + 2, x[step & 1]);
        if (step + 1 < NK) {
          if (i == 0) k_most = f32s::magnitude(k_most, x[(step + 1) & 1]);
          f32s::split_piece(kp[(step + 1) & 1], x[(step + 1) & 1], i);
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
      wait_vmcnt<0>();
    }
    wait_lgkmcnt0();
    fence();
    if (rows_left > SW * SQ) {
      first += SW * SQ;
      rows_left -= SW * SQ;
    } else {
      const int tiles_left = (rows_left + SQ - 1) / SQ;  // of this block, from the tile on: at most SW
      ++k2;
      enter(SW - tiles_left);
    }
    if (k2 <= k1) fetch();
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = (s[r] + small[r]) * prob.c;
    if (rows < SQ) tile::mask_block(rows, hl, s);
    float m_new = m;
#pragma unroll
    for (int r = 0; r < 16; ++r) m_new = fmaxf(m_new, s[r]);
    cur *= prob(m, m_new);
    m = m_new;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r & 3] += prob(s[r], m);
    cur += (sum[0] + sum[1]) + (sum[2] + sum[3]);
    if (k2 != here) {  // the wavefront leaves the block
      const float mb = max_halves(m);
      const float sb = sum_halves(cur * prob(m, mb));
      if (hl == 0) {
        blk_sum(here, wave, n) = sb;
        blk_max(here, wave, n) = mb;
      }
      cur = 0.f;
    }
  }
  m = max_halves(m);
  if (hl == 0) fin_max[wave * SQ + n] = m;
  __syncthreads();

  // Row masses relative to the final maximum, normalised; rows past t_k1 contribute nothing.
  {
    const int row = tid & (SQ - 1);
    float mf = fin_max[row];
#pragma unroll
    for (int w = 1; w < SW; ++w) mf = fmaxf(mf, fin_max[w * SQ + row]);
    for (int j = tid / SQ; j <= k1; j += 64 * SW / SQ) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < SW; ++w) v += blk_sum(j, w, row) * prob(blk_max(j, w, row), mf);
      blk_sum(j, 0, row) = v;
    }
  }
  __syncthreads();
  if (tid < SQ) {
    float l = 0.f;
    for (int j = 0; j <= k1; ++j) l += blk_sum(j, 0, tid);
    row_inv[tid] = tid < q_rows ? 1.f / l : 0.f;
  }
  __syncthreads();
  // One partial per FQ query rows, as the other kernel leaves them.
  const int n_parts = (t_k1 + FQ - 1) / FQ, half = tid / 32, j = tid % 32;  // MAXK is at most 32
  const int part = qt * (SQ / FQ) + half;
  if (half < SQ / FQ && j <= k1 && part < n_parts) {
    float v = 0.f;
#pragma unroll
    for (int rr = 0; rr < FQ; ++rr) v += blk_sum(j, 0, half * FQ + rr) * row_inv[half * FQ + rr];
    job.partial[(static_cast<long long>(bh) * n_parts + part) * p.K + j] = v;
  }
}

// The reductions of a launch's partial sums.  Their bound is the latency of a few dependent reads, so these arguments are a
// short record of their own (a launch reads it cold), in which all that a thread needs is one read away; reads of tiles and
// batch rows go out together.  fp32, 8 heads, batch 2, eight calls of up to 25 tiles each with its reduction: 93 -> 89 us.
struct FinishJob {
  const float* partial;  // [batch*H][n_qtiles][K]
  float* mass;           // [batch*H][K], may be null in the accumulating variant
  int k1, rows;          // query scale, its query rows
};
struct FinishParams {
  int H, batch, K, qpt;  // qpt: query rows per partial sum
  float* beta;           // [L][H][K][K] or null
  float weight;
  int layer;
  FinishJob job[MAXK];
};

__device__ __forceinline__ void touch_params(const FinishParams& p, const FinishJob& job) {
  asm volatile("; kernel arguments" ::"s"(p.H), "s"(p.batch), "s"(p.qpt), "s"(p.layer), "s"(job.partial), "s"(job.mass), "s"(job.k1),
               "s"(job.rows));
}

// Sum of one (batch row, head, key block) entry over the query tiles, in tile order, divided by the number of
// query rows.  The loads of a group of sixteen go out together, past the last tile to its place again; the additions keep the
// order (adding a zero changes no bit: masses are not negative).
__device__ __forceinline__ float tile_sum_in_order(const FinishParams& p, const FinishJob& job, long long bh, int j) {
  constexpr int GROUP = 16;
  if (j > job.k1) return 0.f;
  const int n_qtiles = (job.rows + p.qpt - 1) / p.qpt;
  const float* src = job.partial + bh * n_qtiles * p.K + j;
  float v = 0.f;
  for (int qt = 0; qt < n_qtiles; qt += GROUP) {
    float x[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) x[u] = src[static_cast<long long>(min(qt + u, n_qtiles - 1)) * p.K];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) v += qt + u < n_qtiles ? x[u] : 0.f;
  }
  return v / static_cast<float>(job.rows);
}

// Adds the per-tile partial sums in tile order and divides by the number of query rows.  blockIdx.y = scale of
// the launch.
__global__ void calibrate_finish_kernel(FinishParams p) {
  const FinishJob job = p.job[blockIdx.y];
  touch_params(p, job);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = p.batch * p.H * p.K;
  if (i >= total) return;
  job.mass[i] = tile_sum_in_order(p, job, i / p.K, i % p.K);
}

// Same reduction followed by the dataset average in one pass: eight batch rows of 32 (head, key block) entries side by
// side, added in the order of the rows, so the result has the bits of calibrate_finish_kernel followed by
// accumulate_beta_kernel.
constexpr int FINISH_ENTRIES = 32, FINISH_ROWS = 8;

__global__ __launch_bounds__(FINISH_ENTRIES * FINISH_ROWS) void calibrate_finish_accumulate_kernel(FinishParams p) {
  __shared__ float row_mass[FINISH_ROWS][FINISH_ENTRIES];
  const FinishJob job = p.job[blockIdx.y];
  touch_params(p, job);
  const int column = threadIdx.x % FINISH_ENTRIES, row = threadIdx.x / FINISH_ENTRIES;
  const int i = blockIdx.x * FINISH_ENTRIES + column;
  const bool valid = i < p.H * p.K;
  const int h = i / p.K, j = i % p.K;
  float* const out = p.beta + ((static_cast<long long>(p.layer) * p.H + h) * p.K + job.k1) * p.K + j;
  const bool writes = valid && row == 0;
  const float before = writes ? *out : 0.f;
  float acc = 0.f;
  for (int b0 = 0; b0 < p.batch; b0 += FINISH_ROWS) {
    const int b = b0 + row;
    if (valid && b < p.batch) {
      const long long bh = static_cast<long long>(b) * p.H + h;
      const float v = tile_sum_in_order(p, job, bh, j);
      if (job.mass) job.mass[bh * p.K + j] = v;
      row_mass[row][column] = v;
    }
    __syncthreads();
    if (writes)
      for (int r = 0; r < min(p.batch - b0, FINISH_ROWS); ++r) acc += row_mass[r][column];
    __syncthreads();
  }
  if (writes) *out = before + p.weight * acc;
}

__global__ void accumulate_beta_kernel(int H, int batch, int K, int layer, int k1, const float* mass, float weight,
                                       float* beta) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= H * K) return;
  const int h = i / K, k2 = i % K;
  float v = 0.f;
  for (int b = 0; b < batch; ++b) v += mass[(static_cast<long long>(b) * H + h) * K + k2];
  beta[((static_cast<long long>(layer) * H + h) * K + k1) * K + k2] += weight * v;
}

// Query rows per partial sum.
int queries_per_tile(int dtype) { return dtype == HEATKV_BF16 ? CBM1 : FQ; }

}  // namespace

namespace {

hipError_t launch_calibrate_one_tile(const CalibParams& p, const CalibDirect& direct, int d, size_t lds, hipStream_t stream) {
  const dim3 grid(p.H), block(64 * FW * p.batch);
  if (p.batch == 1) {
    if (d == 64)
      hipLaunchKernelGGL((calibrate_f32_kernel<64, 1>), grid, block, lds, stream, p, direct);
    else
      hipLaunchKernelGGL((calibrate_f32_kernel<128, 1>), grid, block, lds, stream, p, direct);
    return hipGetLastError();
  }
  static_assert(2 * f32_lds_bytes<64>(MAXK - 1) <= 64 * 1024 && f32_lds_bytes<128>(MAXK - 1) <= 64 * 1024,
                "launched without a raised limit");
  // d = 128: more than 64 KB of dynamic LDS needs the function attribute raised, once per device.
  static std::atomic<unsigned long long> raised{0};  // one bit per device ordinal below 64
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !(raised.load(std::memory_order_acquire) >> dev & 1)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&calibrate_f32_kernel<128, 2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(2 * f32_lds_bytes<128>(MAXK - 1)));
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) raised.fetch_or(1ull << dev, std::memory_order_release);
  }
  if (d == 64)
    hipLaunchKernelGGL((calibrate_f32_kernel<64, 2>), grid, block, 2 * lds, stream, p, direct);
  else
    hipLaunchKernelGGL((calibrate_f32_kernel<128, 2>), grid, block, 2 * lds, stream, p, direct);
  return hipGetLastError();
}

}  // namespace

size_t calibrate_workspace_bytes(int dtype, int, int H, int batch, int K, int t_k1) {
  const int qpt = queries_per_tile(dtype);
  const size_t n_qtiles = size_t((t_k1 + qpt - 1) / qpt);
  return size_t(batch) * H * n_qtiles * K * sizeof(float);
}

// Several scales in one launch: each scale's partials start on a 256-byte boundary.
size_t calibrate_scales_workspace_bytes(int dtype, int d, int H, int batch, int K, const int32_t* t, int n_scales,
                                        const int32_t* k1) {
  size_t total = 0;
  for (int i = 0; i < n_scales; ++i)
    total += (calibrate_workspace_bytes(dtype, d, H, batch, K, t[k1[i]]) + 255) / 256 * 256;
  return total;
}

hipError_t launch_calibrate(const CalibrateArgs& a, hipStream_t stream) {
  if (a.n_scales < 1 || a.n_scales > MAXK) return hipErrorInvalidValue;
  CalibParams p{};
  p.H = a.H;
  p.batch = a.batch;
  p.K = a.K;
  p.n_scales = a.n_scales;
  int acc = 0;
  for (int k = 0; k < a.K; ++k) {
    p.t[k] = a.t[k];
    acc += a.t[k];
    p.c[k] = acc;
  }
  p.sm_scale = a.sm_scale;
  const bool bf16 = a.dtype == HEATKV_BF16;
  // bf16: the instance with two query sets per wavefront if its workgroups fill their 512 slots at least once.
  // Both leave one partial per 128 query rows (qpt), bit for bit the same ones.
  const int qpt = queries_per_tile(a.dtype);
  int rows_per_block = qpt;
  if (bf16) {
    unsigned long long wide_blocks = 0;
    for (int i = 0; i < a.n_scales; ++i)
      wide_blocks += (unsigned long long)((a.t[a.k1[i]] + 2 * CBM1 - 1) / (2 * CBM1)) * a.H * a.batch;
    if (wide_blocks >= 512) rows_per_block = 2 * CBM1;
  }
  // The (batch row, head) pairs are padded to a multiple of 8 so that id % 8 is the XCD.
  const unsigned pairs = (unsigned(a.H) * a.batch + 7) / 8 * 8;
  // fp32: the kernel of a scale follows from that scale alone, so that a launch of several has the bits of one each; the scales
  // of either kernel are a launch, and the second one no longer fills the gaps of the first.  Hence only large scales on three
  // bf16 parts (all scales up to the largest in one call, fp32 instructions alone -> both, d = 128): 16 pairs, 400 rows 37 -> 39 us,
  // 48 x 256 40 -> 42, 72 x 256 39 -> 41, 64 x 400 107 -> 109, 64 x 484 140 -> 124, 128 x 256 93 -> 83, 256 x 400 314 -> 291; d = 64, where
  // parts cost as much for half the work: 64 x 400 63 -> 68.  One scale alone, below 256 rows only in few turns (128 pairs, 225 x 633
  // keys, 4 turns 74 -> 64; 384 pairs, 196 x 408, 11 turns 120 -> 124; 625 pairs, 225 x 633, 20 turns 280 -> 289, 324 x 957 540 -> 535).
  // The block sums of many scales (d = 128: more than 15) do not fit next to the key stages.
  auto split_bytes = [&](int k1) { return a.d == 64 ? SplitLds<64>::bytes(k1) : SplitLds<128>::bytes(k1); };
  auto takes_split = [&](int i) {
    const int t = a.t[a.k1[i]];
    const unsigned long long blocks16 = (unsigned long long)((t + FQ - 1) / FQ) * pairs;
    const unsigned long long blocks32 = (unsigned long long)((t + SQ - 1) / SQ) * pairs;
    return !bf16 && split_bytes(a.k1[i]) <= kMaxLds && blocks16 >= (a.d == 64 ? 8192 : 1920) && (t >= 256 || blocks32 <= 7 * 256) &&
           f32s::pays(a.d, t, blocks16, blocks32, a.sm_scale);
  };
  if (bf16 && a.d != 128 && a.d != 64) return hipErrorInvalidValue;
  if (!bf16 && a.d != 64 && a.d != 128) return hipErrorInvalidValue;
  // Largest scale first: its workgroups are the long ones, the short ones then fill the gaps they leave.
  int order[MAXK];
  for (int i = 0; i < a.n_scales; ++i) order[i] = i;
  std::stable_sort(order, order + a.n_scales, [&](int x, int y) { return a.t[a.k1[x]] > a.t[a.k1[y]]; });
  const int n_split = int(std::stable_partition(order, order + a.n_scales, takes_split) - order);
  CalibParams split_p = p;
  split_p.n_scales = n_split;
  p.n_scales = a.n_scales - n_split;
  FinishParams fin{};
  unsigned blocks = 0, split_blocks = 0;
  size_t ws_off = 0;
  int k1_max = 0, split_k1_max = 0;
  for (int i = 0; i < a.n_scales; ++i) {
    const int src = order[i];
    const bool split = i < n_split;
    ScaleJob& job = split ? split_p.job[i] : p.job[i - n_split];
    unsigned& begin = split ? split_blocks : blocks;
    job.k1 = a.k1[src];
    job.block_begin = int(begin);
    job.q = a.q[src];
    job.k_all = a.k_all[src];
    job.partial = reinterpret_cast<float*>(static_cast<char*>(a.ws) + ws_off);
    fin.job[i] = FinishJob{job.partial, a.mass[src], job.k1, a.t[job.k1]};
    const int rows = split ? SQ : rows_per_block;
    begin += unsigned((a.t[job.k1] + rows - 1) / rows) * pairs;
    ws_off += (calibrate_workspace_bytes(a.dtype, a.d, a.H, a.batch, a.K, a.t[job.k1]) + 255) / 256 * 256;
    int& last = split ? split_k1_max : k1_max;
    last = std::max(last, job.k1);
  }
  if (bf16) {
    // Many scales need more than the default 64 KB of dynamic LDS for the parked block sums: raise the limit to
    // what the largest scale count can ask for, once per device.
    static std::atomic<unsigned long long> raised{0};  // one bit per device ordinal below 64
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !(raised.load(std::memory_order_acquire) >> dev & 1)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&calibrate_bf16_kernel<2, 128>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, int(calib_lds_bytes(MAXK - 1, 2, 128)));
      if (e != hipSuccess) return e;
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&calibrate_bf16_kernel<2, 64>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, int(calib_lds_bytes(MAXK - 1, 2, 64)));
      if (e != hipSuccess) return e;
      if (dev >= 0 && dev < 64) raised.fetch_or(1ull << dev, std::memory_order_release);
    }
    const size_t lds_bytes = calib_lds_bytes(k1_max, rows_per_block == CBM1 ? 1 : 2, a.d);
    if (a.d == 128 && rows_per_block == CBM1)
      hipLaunchKernelGGL((calibrate_bf16_kernel<1, 128>), dim3(blocks), dim3(256), lds_bytes, stream, p);
    else if (a.d == 128)
      hipLaunchKernelGGL((calibrate_bf16_kernel<2, 128>), dim3(blocks), dim3(256), lds_bytes, stream, p);
    else if (rows_per_block == CBM1)
      hipLaunchKernelGGL((calibrate_bf16_kernel<1, 64>), dim3(blocks), dim3(256), lds_bytes, stream, p);
    else
      hipLaunchKernelGGL((calibrate_bf16_kernel<2, 64>), dim3(blocks), dim3(256), lds_bytes, stream, p);
  }
  if (n_split > 0) {
    static std::atomic<unsigned long long> raised{0};  // one bit per device ordinal below 64
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !(raised.load(std::memory_order_acquire) >> dev & 1)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&calibrate_f32_split_kernel<64>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&calibrate_f32_split_kernel<128>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
      if (e != hipSuccess) return e;
      if (dev >= 0 && dev < 64) raised.fetch_or(1ull << dev, std::memory_order_release);
    }
    if (a.d == 64)
      hipLaunchKernelGGL(calibrate_f32_split_kernel<64>, dim3(split_blocks), dim3(64 * SW), split_bytes(split_k1_max), stream,
                         split_p);
    else
      hipLaunchKernelGGL(calibrate_f32_split_kernel<128>, dim3(split_blocks), dim3(64 * SW), split_bytes(split_k1_max), stream,
                         split_p);
  }
  if (!bf16 && p.n_scales > 0) {
    const CalibDirect direct{a.mass[0], a.beta, a.weight, a.layer};
    size_t lds = a.d == 64 ? f32_lds_bytes<64>(k1_max) : f32_lds_bytes<128>(k1_max);
    // One query tile and the average asked for: no second launch.  Several scales in one call keep it, the launch reduces all.
    // Two batch rows share a workgroup, two wavefronts per SIMD whose matrix instructions take turns, where the other form has
    // a unit for each (up to 128 heads): every key tile costs more, until the launch is not worth it.  Two -> one launch, 4 to
    // 128 heads, d = 64: 272 keys (17 tiles) 7.5 -> 7.3 us, 384 8.2 -> 8.2, 512 8.9 -> 9.3, 1000 12.5 -> 14.6; d = 128: 64 keys 6.4 ->
    // 6.1, 31 scales of 16 up to 8 tiles 7.8 -> 7.4 and up to 12 8.7 -> 8.8, but 112 + 16 keys 7.4 -> 7.5, 272 9.4 -> 10.7, 1000 17.4 ->
    // 23.3.  129 to 256 heads share units in either form: 160 heads, d = 128, 64 keys 8.0 -> 6.3, 1000 23.5 -> 20.6.
    int key_tiles = 0;
    for (int k = 0; k <= a.k1[0]; ++k) key_tiles += (a.t[k] + FQ - 1) / FQ;
    const bool rows_share = a.batch == 1 || (a.batch == 2 && (key_tiles <= (a.d == 64 ? 20 : 8) || (a.H > 128 && a.H <= 256)));
    if (a.beta && a.n_scales == 1 && a.t[a.k1[0]] <= FQ && rows_share)
      return launch_calibrate_one_tile(p, direct, a.d, lds, stream);
    const int fit = std::min(int(kMaxLds / lds), a.d == 64 ? 7 : 4);
    const int per_unit = rules::calibration_f32_per_unit(a.d, p.n_scales, blocks, fit);
    if (per_unit < fit)  // more LDS than it needs keeps further workgroups off the unit
      lds = std::max(lds, size_t(kMaxLds / (per_unit + 1) + 1024) & ~size_t(1023));
    if (a.d == 64)
      hipLaunchKernelGGL((calibrate_f32_kernel<64, 0>), dim3(blocks), dim3(64 * FW), lds, stream, p, direct);
    else
      hipLaunchKernelGGL((calibrate_f32_kernel<128, 0>), dim3(blocks), dim3(64 * FW), lds, stream, p, direct);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  fin.H = a.H;
  fin.batch = a.batch;
  fin.K = a.K;
  fin.qpt = qpt;
  fin.beta = a.beta;
  fin.weight = a.weight;
  fin.layer = a.layer;
  if (a.beta) {
    hipLaunchKernelGGL(calibrate_finish_accumulate_kernel,
                       dim3((a.H * a.K + FINISH_ENTRIES - 1) / FINISH_ENTRIES, a.n_scales),
                       dim3(FINISH_ENTRIES * FINISH_ROWS), 0, stream, fin);
  } else {
    const int total = a.batch * a.H * a.K;
    hipLaunchKernelGGL(calibrate_finish_kernel, dim3((total + 255) / 256, a.n_scales), dim3(256), 0, stream, fin);
  }
  return hipGetLastError();
}

// Workspace for callers that cannot allocate: the per-tile partial sums live in this file-scope device array
// instead of a caller buffer.  Every GPU the library runs on holds its own copy at its own address until the
// process ends; the array's name is only a host-side handle, the device address comes from
// hipGetSymbolAddress, once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kCalibrateStaticBytes];

hipError_t calibrate_static_workspace(void** ptr) {
  static std::mutex mu;
  static void* per_device[64] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

hipError_t launch_accumulate_beta(int H, int batch, int K, int layer, int k1, const float* mass, float weight,
                                  float* beta, hipStream_t stream) {
  const int total = H * K;
  hipLaunchKernelGGL(accumulate_beta_kernel, dim3((total + 255) / 256), dim3(256), 0, stream, H, batch, K, layer, k1,
                     mass, weight, beta);
  return hipGetLastError();
}

}  // namespace heatkv
