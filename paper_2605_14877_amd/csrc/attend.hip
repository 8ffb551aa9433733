// Next-scale attention over the ragged per-head KV cache (Sec. 3.1 attention rows,
// Sec. 3.3 for which prior scales a head still holds).
//
// For head (b,h) the keys are the head's run of retained rows in the arena
// followed by the t_k rows of the current scale; queries are the t_k rows of
// the current scale.  The kernel walks this virtual key sequence in tiles, keeps
// running row maxima and row sums in fp32 (online softmax) and normalises once at
// the end.  This file holds the bf16 kernel and the launcher; bf16 launches of short walks or few workgroups:
// attend_short.hip; fp32: attend_f32.hip and, for many queries, attend_f32_split.hip.
#include <atomic>
#include <type_traits>

#include "attend_params.h"
#include "device_util.h"
#include "kernels.h"
#include "launch_rules.h"
#include "tile_lds.h"

namespace heatkv {

namespace {

// ---------------------------------------------------------------------------
// bf16, d = 128 or 64: matrix-core kernel (the description takes d = 128: rows of 256 bytes).
//
// Workgroup = 4 wavefronts x 32 queries, two workgroups per compute unit.  The
// keys of a head are walked in 64-row tiles, first the current scale (dense
// tensor), then the head's retained run in the arena (attention does not depend
// on key order, and each segment is then one contiguous range, so a tile's
// addresses are a wavefront-uniform base plus a fixed per-lane offset).
//
// Tiles go from HBM straight into LDS (buffer_load .. lds, no registers, no LDS
// store instructions), double-buffered with one barrier per tile; the descriptor's
// range check takes care of ragged tiles.  A tile is stored row-major, 256 bytes
// per row, unpadded; the 16-byte chunks of a row are XOR-swizzled with the row number (the lane that fills an LDS slot simply
// fetches the matching global chunk), K tiles and V tiles each with the pattern
// that keeps their read instruction free of bank conflicts (tile_lds.h holds the
// format; the calibration kernel and the measurement probes share it).
//
// Scores are produced transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: K
// rows are the A operand straight from LDS, Q stays in registers as the B operand.
// One lane then owns one query column: row maxima and sums are in-register
// reductions plus one exchange between the wavefront halves, and the bf16
// probabilities already sit in the B-operand layout of O^T += V^T P^T.  V^T comes
// out of the row-major V tile with the transposing LDS read; the order of keys
// inside a 16-key MFMA step is permuted identically on both operands.
// ---------------------------------------------------------------------------
constexpr int BM = 128;              // queries per workgroup
constexpr int BN = tile::ROWS;       // keys per tile
constexpr int TILE_BYTES_D128 = tile::BYTES;  // 64 rows x 256 bytes

extern __shared__ __attribute__((aligned(1024))) char attend_dynamic_lds[];

// KS = number of key streams.  KS = 1: the workgroup described above.  KS = 2, for launches that give every
// compute unit at most one workgroup (few heads, small batch; launch_rules.h): 8 wavefronts, one workgroup per unit; wavefronts
// 4-7 take the same 128 queries as 0-3 but every other key tile (stream g walks tiles g, g + 2, ...), each
// stream with its own pair of tile stages (128 KB of dynamic LDS; d = 64: 64 KB), and at the end stream 1 hands its partial
// output, row sums and references to stream 0 through LDS.  The unit then runs two wavefronts per SIMD, as it
// does when two workgroups share it, without a second pass over HBM.
//
// FP8: the arenas hold FP8 E4M3 codes, 128 bytes per row (single-stream instances only).  A tile of the retained run
// lands as it is (8 KB) in a landing buffer behind the tile stages, one for K and one for V, and at the top of the
// step that first needs it the whole workgroup rewrites it as a bf16 tile in its stage (exact: every E4M3 value is
// a bf16 value), with one more barrier; from there on the step is the same.  Current-scale tiles are bf16 and go
// straight to their stage.  80 KB of LDS per workgroup: two workgroups still share a compute unit.
//
// D: head dimension, 128 or 64 (rows of 256 or 128 bytes, tiles of 16 or 8 KB, 8 or 4 MFMA steps per score block and
// 4 or 2 accumulator blocks; one query set and bf16 cache rows only).
//
// QS = 2, for launches that keep every compute unit busy for rounds of long walks: 8 wavefronts, one workgroup
// per unit, 256 queries per workgroup; wavefronts 4-7 take the next 128 queries against the SAME key tiles, which
// all eight wavefronts copy together (two instead of four copies per wavefront and tile).  A K/V tile then enters
// the LDS once per 256 queries instead of once per 128: the copies, which cost the single-set instance 14-18 % of
// its time at these scales whether they come from HBM or from L2, are halved per FLOP.  The two wavefronts of a SIMD
// now pass the same barriers and so run the same part of the step at the same time; that costs nothing because
// every slot of the hand-ordered step below mixes matrix and vector work (with the compiler's own order, score
// MFMAs clustered apart from the exponentials, the same instance gained 1 % instead of 4-6 %).
//
// COPIERS, for launches that give every compute unit at most one workgroup, where two key streams do not pay (launch_rules.h):
// four more wavefronts copy the tiles and do nothing else.  A wavefront that issues copies is held about 100 cycles by each, and here it
// has its SIMD to itself, with nobody to compute meanwhile.  Same steps, same bits as without.
template <int KS, bool FP8, int D, int QS = 1, bool COPIERS = false>
__global__ __launch_bounds__(256 * KS * QS * (COPIERS ? 2 : 1), (KS == 1 && QS == 1) ? 2 : 1) void attend_bf16_kernel(AttendParams p) {
  static_assert(KS == 1 || KS == 2, "one or two key streams");
  static_assert(QS == 1 || QS == 2, "one or two query sets");
  static_assert(!(FP8 && KS == 2), "the 8-bit cache path has one key stream");
  static_assert(D == 128 || (D == 64 && !FP8), "d = 64: bf16 cache rows");
  static_assert(QS == 1 || (KS == 1 && D == 128), "two query sets: single stream, d = 128");
  static_assert(!COPIERS || (KS == 1 && QS == 1), "copying wavefronts: one stream, one query set");
  constexpr int LANES = 256 * KS * QS * (COPIERS ? 2 : 1);  // of the workgroup
  constexpr int NW = 4 * QS;  // wavefronts that share the copying of a tile
  constexpr int ROW_BYTES = 2 * D;            // one bf16 row
  constexpr int TILE_BYTES = BN * ROW_BYTES;  // 16 KB (d = 128) or 8 KB (d = 64)
  constexpr int CPR = ROW_BYTES / 16;         // 16-byte chunks per row
  constexpr int NK = D / 16, NV = D / 32;     // MFMA steps of a score block, accumulator blocks of 32 columns
  constexpr bool kStaticLds = KS == 1 && !FP8;
  __shared__ __attribute__((aligned(1024))) char lds_static[kStaticLds ? 2 : 1][2][kStaticLds ? TILE_BYTES : 16];
  // [stream * 2 + stage][K,V]; 64 KB are static, anything more exceeds the static limit and comes as dynamic LDS
  char(*lds)[2][TILE_BYTES] = kStaticLds ? reinterpret_cast<char(*)[2][TILE_BYTES]>(&lds_static[0][0][0])
                                         : reinterpret_cast<char(*)[2][TILE_BYTES]>(attend_dynamic_lds);
  char* const raw_k = reinterpret_cast<char*>(lds) + 4 * TILE_BYTES;  // FP8 only: landing buffers, 8 KB each
  char* const raw_v = raw_k + tile::RAW8_BYTES;

  touch_params(p);
  if (static_cast<int>(blockIdx.x) >= p.attend_blocks) {  // fused append: a plain row copy by 256 lanes
    const int j = blockIdx.x - p.attend_blocks;
    if constexpr (COPIERS)  // both halves of the workgroup
      copy_rows_block(p.copy, j % p.ndesc, j / p.ndesc, threadIdx.x >> 8, 2);
    else if ((KS == 1 && QS == 1) || threadIdx.x < 256)
      copy_rows_block(p.copy, j % p.ndesc, j / p.ndesc);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform, kept in a scalar register
  const int g = KS == 1 ? 0 : wave_all >> 2;                      // key stream of this wavefront
  const int qs = QS == 1 ? 0 : wave_all >> 2;                     // query set of this wavefront
  const int wave = wave_all & 3;                                  // its place among the four of the stream / set
  const int lw = QS == 1 ? wave : wave_all;                       // its place among the NW that copy a tile
  const int n = lane & 31, hl = lane >> 5;
  const bool computes = !COPIERS || wave_all < 4, copies_tiles = !COPIERS || wave_all >= 4;

  Task task;
  if (!find_task(p, task)) return;
  const int h = task.h, b = task.b, qt = task.qt, n_prior = task.run_len, run_row = task.run_row;

  const int t_k = p.t_k;
  const long long cur_off = (static_cast<long long>(b) * p.H + h) * t_k * D;
  constexpr int PRIOR_ROW_BYTES = FP8 ? tile::RAW8_ROW_BYTES : ROW_BYTES;
  constexpr int PRIOR_TILE_BYTES = BN * PRIOR_ROW_BYTES;
  const long long run_off = (static_cast<long long>(b) * p.arena_tokens + run_row) * PRIOR_ROW_BYTES;
  const char* k_prior = static_cast<const char*>(p.k_arena) + run_off;
  const char* v_prior = static_cast<const char*>(p.v_arena) + run_off;
  const char* k_cur = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.k_cur) + cur_off);
  const char* v_cur = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.v_cur) + cur_off);

  // Q as B operand: lane (n, hl) holds Q[row][16*ks + 8*hl .. +7] for ks = 0..7.
  const int q_row0 = qt * (BM * QS) + qs * BM + wave * 32;  // first query row of this wavefront
  const int q_row = q_row0 + n;
  bf16x8 qreg[NK] = {};
  if (computes) {
    const int ld = q_row < t_k ? q_row : t_k - 1;
    const bf16_t* qp = static_cast<const bf16_t*>(p.q) + cur_off + static_cast<long long>(ld) * D + 8 * hl;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
  }

  // Tile schedule: tiles [0, tiles_cur) cover the current scale, the rest the retained run.
  const int tiles_cur = (t_k + BN - 1) / BN;
  const int tiles_all = tiles_cur + (n_prior + BN - 1) / BN;
  // Step j of stream g works on tile KS j + g; all streams make steps_all steps (the barriers are shared), a
  // stream whose last step has no tile sits it out.
  const int steps_all = (tiles_all + KS - 1) / KS;
  auto has_tile = [&](int j) { return KS == 1 || KS * j + g < tiles_all; };

  // Loader and reader offsets of the shared tile format.  The copy HBM -> LDS is issued as raw instructions
  // (tile::copy_1k_checked): the compiler then does not see an LDS store it would have to
  // order against the tile reads of the other buffer (it would wait for the whole prefetch in the middle of the
  // math).  Ordering is explicit instead: s_waitcnt vmcnt(0) and the workgroup barrier at the top of every step.
  const int ld_off_k = tile::loader_off_k<ROW_BYTES>(lw, lane);
  const int ld_off_v = tile::loader_off_v<ROW_BYTES>(lw, lane);
  const unsigned lds_base = static_cast<unsigned>(reinterpret_cast<unsigned long long>(
      (__attribute__((address_space(3))) char*)(&lds[0][0][0]))) + g * (4 * TILE_BYTES);
  int k_off[NK], v_off[NV];
  tile::reader_off_k<ROW_BYTES>(lane, k_off);
  tile::reader_off_v<ROW_BYTES>(lane, v_off);

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  const float c = p.sm_scale * kLog2e;
  float m_run = lowest_reference(c), l_run = 0.f;
  // The running reference m_run of a row is only raised when the tile maximum exceeds it by more than
  // kSlack in the exponent (base 2): probabilities are then at most 2^kSlack, far inside fp32/bf16 range,
  // the final division by the row sum makes the result independent of the reference, and the expensive
  // rescaling of the accumulators happens a handful of times per row instead of every few tiles.
  constexpr float kSlack = 8.f;
  const float slack_raw = kSlack / c;
  const bf16x2 ones = {static_cast<bf16_t>(1.f), static_cast<bf16_t>(1.f)};

  // ---- software-pipelined tile loop --------------------------------------------------------------
  // Step `it` computes the scores of tile it+1 (matrix cores) while it turns the scores of tile `it` into
  // probabilities (vector ALU) and accumulates P V for tile `it`.  K tiles are therefore fetched one tile
  // further ahead than V tiles: at the top of step `it` the copies K(it+1) and V(it) must have landed.
  // A tile past the walk's end (the one that a stream's last step lacks, or the one after the last) has no valid rows.
  constexpr int CPT = TILE_BYTES / (1024 * NW);  // copies of a tile per wavefront
  struct TileSpan {
    bool prior;
    int local, left;  // tile number inside its segment, rows from its first one to the segment's end
  };
  auto span_of = [&](int j) {
    const int it = KS * j + g;
    const bool prior = it >= tiles_cur;
    const int local = prior ? it - tiles_cur : it;
    return TileSpan{prior, local, (prior ? n_prior : t_k) - local * BN};
  };
  auto source = [&](int j, const char* cur, const char* prior) {
    const TileSpan t = span_of(j);
    return tile::tile_descriptor<ROW_BYTES>((t.prior ? prior : cur) + static_cast<long long>(t.local) * TILE_BYTES, t.left);
  };
  // The same for the steady-state steps, one tile after the other: K and V of the walk's tile j, rows left from it on.
  struct Walk {
    const char *k, *v;
    int it, left;
  };
  auto walk_at = [&](int j) {
    const TileSpan t = span_of(j);
    const long long off = static_cast<long long>(t.local) * TILE_BYTES;
    return Walk{(t.prior ? k_prior : k_cur) + off, (t.prior ? v_prior : v_cur) + off, KS * j + g, t.left};
  };
  auto advance = [&](Walk& w) {
    w.it += KS;
    w.k += KS * TILE_BYTES;
    w.v += KS * TILE_BYTES;
    w.left -= KS * BN;
    const int local = w.it - tiles_cur;
    if (local >= 0 && local < KS) {  // into the retained run
      w.k = k_prior + local * TILE_BYTES;
      w.v = v_prior + local * TILE_BYTES;
      w.left = n_prior - local * BN;
    }
  };
  // Copy i (0 .. CPT - 1) of a tile into K (V) stage `buf`.
  const unsigned lds_wave = lds_base + lw * 1024;
  auto copy_k = [&](const tile::Descriptor& src, int buf, int i) {
    tile::copy_1k_checked(lds_wave, buf * (2 * TILE_BYTES) + i * (1024 * NW), ld_off_k, src, i * (1024 * NW));
  };
  auto copy_v = [&](const tile::Descriptor& src, int buf, int i) {
    tile::copy_1k_checked(lds_wave, buf * (2 * TILE_BYTES) + TILE_BYTES + i * (1024 * NW), ld_off_v, src, i * (1024 * NW));
  };
  auto issue_k = [&](int j, int buf) {
    if constexpr (FP8) {  // codes land in the K landing buffer; the step that needs the tile converts it
      const TileSpan t = span_of(j);
      if (t.prior) {
        tile::issue_raw8<NW>(lds_base + 4 * TILE_BYTES, lw, lane, t.left,
                             k_prior + static_cast<long long>(t.local) * PRIOR_TILE_BYTES);
        return;
      }
    }
    const tile::Descriptor src = source(j, k_cur, k_prior);
#pragma unroll
    for (int i = 0; i < CPT; ++i) copy_k(src, buf, i);
  };
  auto issue_v = [&](int j, int buf) {
    if constexpr (FP8) {
      const TileSpan t = span_of(j);
      if (t.prior) {
        tile::issue_raw8<NW>(lds_base + 4 * TILE_BYTES + tile::RAW8_BYTES, lw, lane, t.left,
                             v_prior + static_cast<long long>(t.local) * PRIOR_TILE_BYTES);
        return;
      }
    }
    const tile::Descriptor src = source(j, v_cur, v_prior);
#pragma unroll
    for (int i = 0; i < CPT; ++i) copy_v(src, buf, i);
  };

  // S^T = K Q^T for the 64 keys of the K tile in buffer `buf` x this wavefront's 32 queries.
  // s[cb][r] is key 32*cb + 8*(r/4) + 4*hl + r%4 of the tile, query column n.
  auto scores = [&](f32x16 (&s)[2], auto buf_tag) {
    constexpr int buf = decltype(buf_tag)::value;
    const char* kt = lds[2 * g + buf][0];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[cb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kt + cb * 32 * ROW_BYTES + k_off[ks]);
        s[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s[cb], 0, 0, 0);
      }
  };
  // Folds the maximum of a tile's scores (this lane's 32 of them) into the running reference and, rarely,
  // rescales what has been accumulated so far.
  auto raise = [&](float mx) {
    mx = max_halves(mx);
    if (__any(mx > m_run + slack_raw)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = fast_exp2((m_run - m_new) * c);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] *= alpha;
    }
  };
  auto lane_max = [&](const f32x16 (&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[cb][r]);
    return mx;
  };
  // Masks the ragged tail of a tile with `left` rows from its first one on (keys past the end of the scale or of the run
  // get -inf); returns whether there was one.
  auto mask_tail = [&](int left, f32x16 (&s)[2]) {
    if (left >= BN) return false;  // workgroup-uniform and rare: kept a branch
    tile::mask_rows(left, hl, s);
    return true;
  };
  // Masks the tail of tile j and folds its row maxima into the running reference.
  auto settle = [&](int j, f32x16 (&s)[2]) {
    mask_tail(span_of(j).left, s);
    raise(lane_max(s));
  };
  // P^T = 2^(S^T c - m c) in bf16, 16 keys at a time, each chunk feeding O^T += V^T P^T at once.  The row
  // sum is taken over the rounded probabilities, pairwise, with the bf16 dot-product instruction.
  union VOperand {
    struct {
      s16x4 lo, hi;
    } s;
    bf16x8 v;
  };
  auto accumulate = [&](const f32x16 (&s)[2], auto buf_tag) {
    constexpr int buf = decltype(buf_tag)::value;
    const char* vt = lds[2 * g + buf][1];
    const float mc = m_run * c;
#pragma unroll
    for (int chunk = 0; chunk < 4; ++chunk) {
      const int cb = chunk >> 1, ks = chunk & 1;
      VOperand va[NV];
#pragma unroll
      for (int dblk = 0; dblk < NV; ++dblk) {
        const char* base = vt + 16 * chunk * ROW_BYTES + v_off[dblk];
        va[dblk].s.lo = lds_read_tr16(reinterpret_cast<const bf16_t*>(base));
        va[dblk].s.hi = lds_read_tr16(reinterpret_cast<const bf16_t*>(base + 8 * ROW_BYTES));
      }
      union {
        bf16x8 v;
        bf16x2 h[4];
      } pb;
#pragma unroll
      for (int j = 0; j < 8; ++j) pb.v[j] = static_cast<bf16_t>(fast_exp2(fmaf(s[cb][8 * ks + j], c, -mc)));
#pragma unroll
      for (int j = 0; j < 4; ++j) l_run = __builtin_amdgcn_fdot2_f32_bf16(pb.h[j], ones, l_run, false);
#pragma unroll
      for (int dblk = 0; dblk < NV; ++dblk)
        o[dblk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[dblk].v, pb.v, o[dblk], 0, 0, 0);
    }
  };

  // The steady-state step in one piece: scores of the next tile into s_out, P V of this tile from s_in, with the
  // order of issue fixed by hand.  Left to itself the compiler clusters the score MFMAs at the K reads that feed
  // them, back to back, and the exponentials elsewhere; a wavefront issues in order, so an MFMA waiting for the
  // matrix pipe holds back the vector work that could run in the shadow of the one before.  Here the step is a
  // sequence of 32 slots, one MFMA each followed by its share of vector and LDS work; scheduling fences keep the
  // slots apart and the MFMA at the head of its slot:
  //   S(g), g = 0..3: the NK/4 K-steps of the score product that go with chunk g (both 32-key blocks)
  //   A(g): P V for the 16 keys of chunk g (NV MFMAs)
  //   order S(0) A(0) S(1) A(1) S(2) A(2) S(3) A(3).  P(0) is computed in the slots of S(0), P(g+1) in those of
  //   A(g) and S(g+1), the row maxima of the new scores in those of A(3); the K operands of S(g+1) are read in the
  //   slots of S(g), the V operands of A(g+1) in those of A(g): every operand a whole phase before its MFMA (those
  //   of S(0) and A(0), which only exist after the barrier, in preload() and in the slots of S(0)).
  // The step's tile copies go out one per slot, from the second slot on.  The path into LDS takes 64 bytes per clock
  // and compute unit, 512 cycles for a K and a V tile; issued together behind the barrier (by in-kernel clock stamps 550
  // cycles of every step for a lone wavefront, 740 with two workgroups on the unit) they held back the step's arithmetic.  Spread out: t_k = 4096 of
  // the serving shape 4211 -> 4052 us, 1600: 782 -> 751; two key streams at 1024 tokens (batch 2): 56.5 -> 50.6 us.
  // Where they start (slot 0, 1, 2 or 4) and whether every slot or every second one has a copy makes no difference.
  // Returns this lane's maximum over the new scores (before any tail mask).
  auto step_math = [&](const f32x16 (&s_in)[2], f32x16 (&s_out)[2], const bf16x8 (&k0)[2], auto kb1, auto vb0,
                       auto copies, const tile::Descriptor& k_src, const tile::Descriptor& v_src) {
    constexpr int COPIES = decltype(copies)::value * CPT;  // 0: none, 1: the K tile's, 2: those of K and V
    constexpr int KPC = NK / 4;          // K-steps per phase S
    constexpr int NS = 2 * KPC;          // slots of a phase S
    constexpr int NA = NV;               // slots of a phase A
    constexpr int HALVES = 8;            // a chunk's probabilities come in 8 half units (one probability per lane each)
    static_assert(HALVES % NS == 0 && HALVES % (NS + NA) == 0, "phases divide the vector work evenly");
    static_assert(NS == NA, "one V block of A(0) is read per slot of S(0)");
    const char* kt = lds[2 * g + decltype(kb1)::value][0];
    const char* vt = lds[2 * g + decltype(vb0)::value][1];
    const float mc = m_run * c;
    bf16x8 kop[NK][2], vop[4][NV];
    float e[4][8];
    union {
      bf16x8 v;
      bf16x2 h[4];
    } pb[4];
    auto load_k = [&](int ks, int cb) {
      kop[ks][cb] = *reinterpret_cast<const bf16x8*>(kt + cb * 32 * ROW_BYTES + k_off[ks]);
    };
    auto load_v = [&](int chunk, int dblk) {
      const char* base = vt + 16 * chunk * ROW_BYTES + v_off[dblk];
      VOperand t;
      t.s.lo = lds_read_tr16(reinterpret_cast<const bf16_t*>(base));
      t.s.hi = lds_read_tr16(reinterpret_cast<const bf16_t*>(base + 8 * ROW_BYTES));
      vop[chunk][dblk] = t.v;
    };
    // Half unit u (0..7) of chunk `chunk`: one probability per lane; the odd ones also pack a pair and add it to
    // the row sum.
    auto p_half = [&](int chunk, int u) {
      const int cb = chunk >> 1, r = 8 * (chunk & 1) + u;
      e[chunk][u] = fast_exp2(fmaf(s_in[cb][r], c, -mc));
      if (u & 1) {
        pb[chunk].h[u >> 1] = bf16x2{static_cast<bf16_t>(e[chunk][u - 1]), static_cast<bf16_t>(e[chunk][u])};
        l_run = __builtin_amdgcn_fdot2_f32_bf16(pb[chunk].h[u >> 1], ones, l_run, false);
      }
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s_out[cb][r] = 0.f;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) kop[0][cb] = k0[cb];
    float mx = -INFINITY;
    int slot_no = 0;  // compile-time after unrolling
    auto copy_slot = [&] {  // one of the step's tile copies
      const int i = slot_no - 1;
      if (i >= 0 && i < COPIES) {
        if (i < CPT)
          copy_k(k_src, decltype(vb0)::value, i);  // K(j+2): the stage that step j-1 read
        else
          copy_v(v_src, decltype(kb1)::value, i - CPT);  // V(j+1) likewise
      }
      ++slot_no;
    };
    auto s_slot = [&](int gch, int i, int halves_chunk, int& half) {  // slot i of phase S(gch)
      const int ks = gch * KPC + (i >> 1), cb = i & 1;
      s_out[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[ks][cb], qreg[ks], s_out[cb], 0, 0, 0);
      fence();
      if (gch == 0) {  // the rest of this phase's K operands, and the V operands of A(0)
        if (ks + 1 < KPC) load_k(ks + 1, cb);
        load_v(0, i);
      }
      if (gch < 3) load_k(ks + KPC, cb);
      copy_slot();
      const int n = gch == 0 ? HALVES / NS : HALVES / (NS + NA);
      for (int u = 0; u < n; ++u) p_half(halves_chunk, half++);
      fence();
    };
    int half = 0;
#pragma unroll
    for (int i = 0; i < NS; ++i) s_slot(0, i, 0, half);
#pragma unroll
    for (int gch = 0; gch < 4; ++gch) {
      half = 0;
#pragma unroll
      for (int d = 0; d < NA; ++d) {  // slot d of phase A(gch)
        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[gch][d], pb[gch].v, o[d], 0, 0, 0);
        fence();
        if (gch < 3) {
          load_v(gch + 1, d);
          copy_slot();
#pragma unroll
          for (int u = 0; u < HALVES / (NS + NA); ++u) p_half(gch + 1, half++);
        } else {  // the new scores are complete: their maxima, 32 / NA registers per slot
#pragma unroll
          for (int r = d * (32 / NA); r < (d + 1) * (32 / NA); ++r) mx = fmaxf(mx, s_out[r >> 4][r & 15]);
          asm volatile("" : "+v"(mx));  // keeps the partial maximum in this slot (it is only consumed on one branch later)
        }
        fence();
      }
      if (gch < 3) {
#pragma unroll
        for (int i = 0; i < NS; ++i) s_slot(gch + 1, i, gch + 1, half);
      }
    }
    return mx;
  };
  // The K operands of a step's first two MFMAs: read right after the barrier.  Only those: right after a
  // barrier all wavefronts of the workgroup read at once, and what they ask for queues up in front of the first
  // MFMA; everything else is read from the slots of phase S(0) on.
  auto preload = [&](bf16x8 (&k0)[2], auto kb1) {
    const char* kt = lds[2 * g + decltype(kb1)::value][0];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) k0[cb] = *reinterpret_cast<const bf16x8*>(kt + cb * 32 * ROW_BYTES + k_off[0]);
  };

  f32x16 s_cur[2], s_nxt[2];
  // A wavefront whose 32 query rows all lie past t_k (ragged last query tile) keeps loading its share of
  // every tile and keeps the barriers, but leaves the matrix cores to the other workgroup on the unit.
  const bool active = computes && q_row0 < t_k;
  // Steady-state step j (j + 1 < steps_all): K of the stream's tile j+1 sits in K stage kb1, V of its tile j in
  // V stage vb0.  s_in holds the scores of tile j, s_out receives those of tile j+1: the two register sets swap
  // roles from step to step instead of being copied.  With two streams the second may lack the last successor tile: it
  // lands as zeros and is masked like any other ragged tile.  `copies` as for step_math.
  Walk w = walk_at(1);
  auto pipe_step = [&](int j, auto kb1, auto vb0, f32x16 (&s_in)[2], f32x16 (&s_out)[2], auto copies, auto may_be_codes) {
    constexpr int COPIES = decltype(copies)::value;
    constexpr bool CODES = FP8 && decltype(may_be_codes)::value;
    // w: tile j+1 on entry, tile j+2 on return (not kept up where tiles may be codes)
    const int left1 = CODES ? span_of(j + 1).left : w.left;
    tile::Descriptor k_src{}, v_src{};
    if constexpr (!CODES) {
      if constexpr (COPIES > 1) v_src = tile::tile_descriptor<ROW_BYTES>(w.v, w.left);
      advance(w);
      k_src = tile::tile_descriptor<ROW_BYTES>(w.k, w.left);
    }
    wait_vmcnt<0>();
    __syncthreads();
    if constexpr (CODES) {
      // What this step reads and arrived as codes: K(j+1), fetched during step j-1 into the K landing buffer, and
      // V(j) likewise.  Their stages are free (last read in step j-2), the landing buffers are free again after
      // the barrier, before this step's copies go out.
      const bool ck = j + 1 < tiles_all && j + 1 >= tiles_cur, cv = j >= tiles_cur;
      if (ck) tile::convert_raw8<false, LANES>(raw_k, lds[decltype(kb1)::value][0], tid);
      if (cv) tile::convert_raw8<true, LANES>(raw_v, lds[decltype(vb0)::value][1], tid);
      if (ck || cv) __syncthreads();
    }
    bf16x8 k0[2];
    if (active) preload(k0, kb1);
    if constexpr (CODES) {
      if (copies_tiles && j + 2 < steps_all) issue_k(j + 2, decltype(vb0)::value);
      if (copies_tiles && COPIES > 1) issue_v(j + 1, decltype(kb1)::value);
      if (!active) return;
    } else if (!active) {
      if (!copies_tiles) return;
#pragma unroll
      for (int i = 0; i < COPIES * CPT; ++i)
        i < CPT ? copy_k(k_src, decltype(vb0)::value, i) : copy_v(v_src, decltype(kb1)::value, i - CPT);
      return;
    }
    const float mx = step_math(s_in, s_out, k0, kb1, vb0, std::integral_constant<int, CODES || COPIERS ? 0 : COPIES>{}, k_src, v_src);
    raise(mask_tail(left1, s_out) ? lane_max(s_out) : mx);
  };

  // Prologue: all four tile stages are free, so K(0), V(0), K(1) and V(1) all go out at once: one memory round
  // trip before the loop, and a walk of two tiles (every scale of up to 64 tokens) never waits for memory again.
  // Loads return in issue order, so waiting until only the copies younger than K(0) are outstanding means that
  // K(0) has landed (CPT copies per wavefront and bf16 tile, two per 8-bit tile); tile 0 is a current-scale tile,
  // whose address does not depend on the head's run.
  if (!copies_tiles) {
    // the copying wavefronts wait for K(0) before the barrier
  } else if (KS == 1) {
    issue_k(0, 0);
    issue_v(0, 0);
    if (tiles_all > 1) {
      issue_k(1, 1);
      issue_v(1, 1);
      if (FP8 && tiles_cur == 1)  // tile 1 arrives as codes: 8 / NW copies per wavefront for each of K(1), V(1)
        wait_vmcnt<CPT + 2 * (8 / NW)>();
      else
        wait_vmcnt<3 * CPT>();
    } else {
      wait_vmcnt<CPT>();
    }
  } else {
    issue_k(0, 0);
    issue_k(1, 1);
    issue_v(0, 0);
    wait_vmcnt<0>();
  }
  __syncthreads();
  if (active && has_tile(0)) {
    scores(s_cur, std::integral_constant<int, 0>{});
    settle(0, s_cur);
  }
  // Every path reaches the loop through a full wait that the compiler sees (a wavefront that skipped the scores
  // above never waited for its query rows): otherwise it waits for them inside every step, and with them for the
  // tile copies that the step has just issued.  The first step starts with the same wait, so this one is free.
  wait_vmcnt<0>();
  // Scores of even steps live in s_cur, of odd steps in s_nxt.  With one key stream the prologue has fetched V(1): the
  // first step copies K(2) only.
  using Zero = std::integral_constant<int, 0>;
  using One = std::integral_constant<int, 1>;
  using Both = std::integral_constant<int, 2>;
  int it = 0;
  if (steps_all > 1) {
    pipe_step(0, One{}, Zero{}, s_cur, s_nxt, std::integral_constant<int, KS == 1 ? 1 : 2>{}, std::true_type{});
    it = 1;
    if constexpr (FP8) {
      // Steps that touch tiles of the current scale only (K(it+3) at most): the bf16 cache's step, one copy per slot and no
      // test for codes.  At 20x these are nine in ten steps of a large scale, and with their copies in one burst they held
      // the instance back: two layers of 16 heads, batch 32, 13 scales 14378 -> 13998 us (bf16 cache: 13640).
      w = walk_at(2);
      for (; it + 3 < tiles_cur; it += 2) {
        pipe_step(it, Zero{}, One{}, s_nxt, s_cur, Both{}, std::false_type{});
        pipe_step(it + 1, One{}, Zero{}, s_cur, s_nxt, Both{}, std::false_type{});
      }
    }
    for (; it + 2 < steps_all; it += 2) {
      pipe_step(it, Zero{}, One{}, s_nxt, s_cur, Both{}, std::true_type{});
      pipe_step(it + 1, One{}, Zero{}, s_cur, s_nxt, Both{}, std::true_type{});
    }
    if (it + 1 < steps_all) {
      pipe_step(it, Zero{}, One{}, s_nxt, s_cur, Both{}, std::true_type{});
      ++it;
    }
  }
  // Epilogue: the last tile has scores but no successor.
  wait_vmcnt<0>();
  __syncthreads();
  if constexpr (FP8) {
    if (it >= tiles_cur) {  // V of the last tile is still in its landing buffer
      if (it & 1)
        tile::convert_raw8<true, LANES>(raw_v, lds[1][1], tid);
      else
        tile::convert_raw8<true, LANES>(raw_v, lds[0][1], tid);
      __syncthreads();
    }
  }
  if (KS == 1 && QS == 1 && !active) return;
  if (active && has_tile(it)) {
    if (it & 1)
      accumulate(s_nxt, std::integral_constant<int, 1>{});
    else
      accumulate(s_cur, std::integral_constant<int, 0>{});
  }
  if constexpr (QS == 2) {  // the eight output tiles are staged over all four tile buffers: the V tiles must be done with
    __syncthreads();
    if (!active) return;
  }
  if constexpr (KS == 2) {
    // Stream 1 parks its accumulators (64 registers, one 256-byte row of LDS per register), row-sum partials and
    // references in the idle tile stages (66 KB from byte 48 K on: clear of the 16 KB at 0 and at 32 K where
    // stream 0 stages its output; d = 64: 32 registers, 34 KB from byte 24 K on, clear of 8 KB at 0 and at 16 K);
    // stream 0 brings both halves to the larger reference and adds.
    __syncthreads();  // every wavefront has finished reading the tile stages
    float* park = reinterpret_cast<float*>(lds[1][1]) + wave * ((16 * NV + 2) * 64);
    if (g == 1 && active) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) park[(16 * i + r) * 64 + lane] = o[i][r];
      park[16 * NV * 64 + lane] = m_run;
      park[(16 * NV + 1) * 64 + lane] = l_run;
    }
    __syncthreads();
    if (g == 1 || !active) return;
    const float m_other = park[16 * NV * 64 + lane], l_other = park[(16 * NV + 1) * 64 + lane];
    const float m_new = fmaxf(m_run, m_other);
    const float a0 = fast_exp2((m_run - m_new) * c), a1 = fast_exp2((m_other - m_new) * c);  // no tile: lowest reference, factor 0
    l_run = l_run * a0 + l_other * a1;
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][r] = o[i][r] * a0 + park[(16 * i + r) * 64 + lane] * a1;
  }

  const float l_tot = sum_halves(l_run);
  const float inv = 1.f / l_tot;
  // Output through LDS.  A lane owns one query row but only 4 consecutive columns at a time, so direct stores
  // would be 8-byte pieces scattered over 32 rows.  The K buffers are idle by now (their last reader passed the
  // barrier above and no copy is in flight), so every wavefront stages its 32 x d tile in half a K stage, with the
  // 16-byte chunks XORed with the row number, and writes it out as whole rows, 1 KB per instruction.
  char* stage = QS == 1 ? lds[wave >> 1][0] + (wave & 1) * (32 * ROW_BYTES)
                        : reinterpret_cast<char*>(lds) + wave_all * (32 * ROW_BYTES);
  // The lane numbers used from here on are formed anew from the work-item id, hidden from the optimiser, so that
  // they are not kept in registers (or spilled) across the tile loop, which has none to spare.
  int tid_o = threadIdx.x;
  asm volatile("" : "+v"(tid_o));
  const int lane_o = tid_o & 63, n_o = lane_o & 31, hl_o = lane_o >> 5;
#pragma unroll
  for (int dblk = 0; dblk < NV; ++dblk)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = static_cast<bf16_t>(o[dblk][4 * g + e] * inv);
      *reinterpret_cast<bf16x4*>(stage + n_o * ROW_BYTES + (((4 * dblk + g) ^ (n_o & (CPR - 1))) << 4) + 8 * hl_o) = v;
    }
  const int out_row0 = q_row0;
  bf16_t* op = static_cast<bf16_t*>(p.out) + cur_off + static_cast<long long>(out_row0) * D;
  constexpr int ROWS_PER_STORE = 64 / CPR;  // CPR lanes write one row
#pragma unroll
  for (int r = 0; r < 32 / ROWS_PER_STORE; ++r) {
    const int row = ROWS_PER_STORE * r + lane_o / CPR, slot = lane_o & (CPR - 1);
    const uint4 v = *reinterpret_cast<const uint4*>(stage + row * ROW_BYTES + ((slot ^ (row & (CPR - 1))) << 4));
    if (out_row0 + row < t_k) *reinterpret_cast<uint4*>(op + row * D + slot * 8) = v;
  }
}

}  // namespace

size_t attend_workspace_bytes(int, int, int, int, int, int) { return 0; }

namespace {

constexpr int TWO_STREAM_LDS_BYTES = 2 * 2 * 2 * TILE_BYTES_D128;  // two streams x two stages x (K, V)
constexpr int FP8_LDS_BYTES = 2 * 2 * TILE_BYTES_D128 + 2 * tile::RAW8_BYTES;  // two stages x (K, V) + two landing buffers
constexpr int TWO_STREAM_MAX_BLOCKS = 256;                    // compute units of the chip
// Two query sets per workgroup: from this scale size on, when the launch still gives every compute unit two rounds
// of such workgroups (measured: a single round of 256 is slower than 512 workgroups of 128 queries), and when the
// last 256-query tile is not mostly empty (1600 tokens: 7 tiles, the last one a quarter full, measured slower).
constexpr int TWO_SET_MIN_TOKENS = 1024;
constexpr int TWO_SET_MIN_BLOCKS = 512;

// More than 64 KB of dynamic LDS needs the function attribute raised, once per device.
hipError_t allow_lds() {
  static std::atomic<unsigned long long> done{0};  // one bit per device ordinal below 64
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 64 && (done.load(std::memory_order_acquire) >> dev & 1)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bf16_kernel<2, false, 128>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, TWO_STREAM_LDS_BYTES);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bf16_kernel<1, true, 128>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FP8_LDS_BYTES);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bf16_kernel<1, true, 128, 1, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FP8_LDS_BYTES);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bf16_kernel<1, true, 128, 2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, FP8_LDS_BYTES);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bf16_kernel<2, false, 64>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, TWO_STREAM_LDS_BYTES / 2);
  if (e == hipSuccess) e = attend_short_prepare();
  if (e == hipSuccess && dev >= 0 && dev < 64) done.fetch_or(1ull << dev, std::memory_order_release);
  return e;
}

}  // namespace

hipError_t attend_prepare_device(int dtype) { return dtype == HEATKV_BF16 ? allow_lds() : attend_f32_split_prepare(); }

hipError_t launch_attend(const AttendArgs& a, hipStream_t stream) {
  AttendParams p{};
  p.H = a.H;
  p.batch = a.batch;
  p.t_k = a.t_k;
  p.arena_tokens = a.arena_tokens;
  p.work = a.work;
  p.uniform_len = a.uniform_len;
  p.uniform_row0 = a.uniform_row0;
  p.q = a.q;
  p.k_cur = a.k_cur;
  p.v_cur = a.v_cur;
  p.k_arena = a.k_arena;
  p.v_arena = a.v_arena;
  p.out = a.out;
  p.sm_scale = a.sm_scale;
  p.ndesc = a.ndesc;
  unsigned copy_blocks = 0;
  if (a.ndesc > 0) {
    if (a.row_bytes % 16 != 0) return hipErrorInvalidValue;
    p.copy.chunks_per_row = a.row_bytes / 16;
    p.copy.kv_fp8 = a.kv_fp8 ? 1 : 0;
    p.copy.H = a.H;
    p.copy.t_k = a.t_k;
    p.copy.arena_tokens = a.arena_tokens;
    p.copy.descs = a.descs;
    p.copy.k_new = static_cast<const uint4*>(a.k_cur);
    p.copy.v_new = static_cast<const uint4*>(a.v_cur);
    p.copy.k_arena = static_cast<uint4*>(a.k_arena_rw);
    p.copy.v_arena = static_cast<uint4*>(a.v_arena_rw);
    copy_blocks = unsigned(a.ndesc) * a.batch;
  }
  if (a.dtype == HEATKV_BF16) {
    if (a.d != 128 && a.d != 64) return hipErrorInvalidValue;
    if (a.d == 64 && a.kv_fp8) return hipErrorInvalidValue;
    const unsigned pairs8 = (unsigned(a.H) * a.batch + 7) / 8 * 8;  // padded so that id % 8 is the XCD
    // Long walks on a full chip: 256 queries per workgroup share every K/V tile (d = 128, either cache format).
    const int wide = (a.t_k + 2 * BM - 1) / (2 * BM);
    const bool two_sets = a.d == 128 && a.t_k >= TWO_SET_MIN_TOKENS &&
                          unsigned(wide) * pairs8 >= unsigned(TWO_SET_MIN_BLOCKS) && (wide * 2 * BM - a.t_k) * 16 <= a.t_k;
    const unsigned wide_blocks = unsigned(wide) * pairs8;
    auto set_split = [&](int n_qtiles) {
      p.n_qtiles = n_qtiles;
      p.attend_blocks = int(unsigned(n_qtiles) * pairs8);
      p.div_qtiles = reciprocal(p.attend_blocks, n_qtiles);
    };
    set_split((a.t_k + BM - 1) / BM);
    p.div_batch = reciprocal(pairs8, a.batch);
    const dim3 grid(unsigned(p.attend_blocks) + copy_blocks);
    if (!a.kv_fp8 && attend_short_fits(p, a.d, a.max_len, copy_blocks)) {
      const hipError_t e = allow_lds();
      return e == hipSuccess ? launch_attend_short(p, a.d, a.max_len, copy_blocks, stream) : e;
    }
    // At most one workgroup per compute unit: two key streams per workgroup put two wavefronts on every SIMD.
    const unsigned tiles = (a.t_k + BN - 1) / BN + (a.max_len + BN - 1) / BN, with_queries = unsigned(p.n_qtiles) * a.H * a.batch;
    const bool two_streams = !a.kv_fp8 && p.attend_blocks <= TWO_STREAM_MAX_BLOCKS && a.t_k >= TWO_STREAM_MIN_TOKENS &&
                             rules::two_key_streams(a.d, with_queries, unsigned(a.update_descs) * a.batch, tiles);
    // Otherwise wavefronts that only copy (112 workgroups of 784 tokens, two streams -> copiers: d = 128 23.9 us -> 24.1, d = 64 17.0
    // -> 18.6).  8-bit cache rows have one stream, hence copiers for walks of any length.
    const bool copiers = !two_streams && p.attend_blocks <= TWO_STREAM_MAX_BLOCKS &&
                         rules::copying_wavefronts(a.d, with_queries, copy_blocks, tiles);
    if (a.d == 64 && two_streams) {
      const hipError_t e = allow_lds();
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((attend_bf16_kernel<2, false, 64>), grid, dim3(512), TWO_STREAM_LDS_BYTES / 2, stream, p);
    } else if (copiers && !a.kv_fp8) {
      if (a.d == 64)
        hipLaunchKernelGGL((attend_bf16_kernel<1, false, 64, 1, true>), grid, dim3(512), 0, stream, p);
      else
        hipLaunchKernelGGL((attend_bf16_kernel<1, false, 128, 1, true>), grid, dim3(512), 0, stream, p);
    } else if (a.d == 64) {  // rows of 128 bytes
      hipLaunchKernelGGL((attend_bf16_kernel<1, false, 64>), grid, dim3(256), 0, stream, p);
    } else if (a.kv_fp8) {  // 8-bit cache rows: the single-stream instances with landing buffers
      const hipError_t e = allow_lds();
      if (e != hipSuccess) return e;
      if (two_sets) {
        set_split(wide);
        hipLaunchKernelGGL((attend_bf16_kernel<1, true, 128, 2>), dim3(wide_blocks + copy_blocks), dim3(512),
                           FP8_LDS_BYTES, stream, p);
      } else {
        if (copiers)
          hipLaunchKernelGGL((attend_bf16_kernel<1, true, 128, 1, true>), grid, dim3(512), FP8_LDS_BYTES, stream, p);
        else
          hipLaunchKernelGGL((attend_bf16_kernel<1, true, 128>), grid, dim3(256), FP8_LDS_BYTES, stream, p);
      }
    } else if (two_streams) {
      const hipError_t e = allow_lds();
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((attend_bf16_kernel<2, false, 128>), grid, dim3(512), TWO_STREAM_LDS_BYTES, stream, p);
    } else if (two_sets) {
      set_split(wide);
      hipLaunchKernelGGL((attend_bf16_kernel<1, false, 128, 2>), dim3(wide_blocks + copy_blocks), dim3(512), 0, stream, p);
    } else {
      hipLaunchKernelGGL((attend_bf16_kernel<1, false, 128>), grid, dim3(256), 0, stream, p);
    }
  } else {
    if (a.kv_fp8) return hipErrorInvalidValue;
    return launch_attend_f32(p, a.d, copy_blocks, stream);
  }
  return hipGetLastError();
}

}  // namespace heatkv
