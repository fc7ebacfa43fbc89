// Register-streaming MFMA kernels for O = W_s x I (Section 5, "GPU
// Implementation"): the fp32 kernel, and the launcher and device tables of both
// dtypes (the bf16 kernel is in rbgp_reg_bf16_kernel.h).
//
// Work decomposition.  One wavefront owns: a cluster of U tile rows u_o, one G_i
// vertex u_i (so, per tile row, the R = |G_r.U|*|G_b.U| rows that share a column
// set: row repetition, Section 5) and 64 columns of O.  It walks the union of the
// cluster's nonzero tiles (tile skipping through G_o's adjacency, Section 5)
// stage by stage; a stage is VC columns of G_r of one tile.  The rows of I a stage
// touches are loaded straight from global memory into VGPRs and each loaded row
// is used for every tile row of the cluster that has the tile: the register-level
// reuse the paper obtains from row repetition, extended across tile rows.  No
// LDS, no barrier in the main loop: waves are independent; loads are issued one
// stage ahead (two or four in the variants with several register sets), slot by
// slot, into the registers the previous MFMAs just released, and the compiler's
// vmcnt bookkeeping provides the software pipeline.  (LDS is
// used once, after the loop, when the stage list of a cluster is split over
// several waves for small N.)
// The same kernel serves the fused 3x3 convolution: only the addresses of the
// loads differ (see `off` in the prologue).
//
// Arithmetic.  v_mfma_f32_16x16x1_4b_f32: four independent 16x16 outer products
// per instruction.  The 64 lanes form 4 groups of 16 (= the 4 blocks).  One
// 16-byte-per-lane load (a "slot") brings 4 rows of I x 64 columns: group g reads
// contraction step 4*o + g of the stage, lane j of the group columns 4j..4j+3.
// Block g multiplies its row of I by the weights of that contraction step for 16
// weight rows: 16/RS tile rows of the cluster (RS = R rounded up to a power of
// two) that share the tile, RS rows each; a tile row that lacks the tile
// contributes zeros.  The four blocks thus accumulate different contraction steps
// of the same 16 x 16 outputs in different accumulator registers, which are
// added in the epilogue.  The 4x4x1 form would multiply no structural zero, but
// one wave per SIMD cannot issue it fast enough (measured: 8-cycle instructions
// issue every 13 cycles and every other instruction costs an issue slot too); the
// 32-cycle 16x16x1 form hides the whole instruction stream behind the matrix core.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <type_traits>
#include <vector>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"

#define RBGP_HIP(call)                                                          \
  do {                                                                          \
    hipError_t e_ = (call);                                                     \
    if (e_ != hipSuccess) {                                                     \
      char buf_[256];                                                           \
      std::snprintf(buf_, sizeof buf_, "%s: %s", #call, hipGetErrorString(e_)); \
      rbgp_set_hip_error(buf_);                                                 \
      return RBGP_EHIP;                                                         \
    }                                                                           \
  } while (0)

using namespace rbgp_reg;

namespace {

// KC: contraction steps per stage; RS: weight rows per tile row in the 16-row MFMA group
// (cluster size MG = 16 / RS).  The weights stream from global memory like I (they are L2 hits).
// TAPS (fused 3x3 convolution on a tap-grouped layout, image width dividing 64): slots 3p,
// 3p+1, 3p+2 of a lane group are the taps dx = -1, 0, +1 of one (channel, dy) pair, i.e. three
// windows of the same pixel row shifted by one pixel.  Only the middle one is loaded; the other
// two are put together from it and the neighbouring lane's pixel (DPP), zero at an image border.
// Stages of 8 steps make short waves (a transposed 3x3 layer: 64 MFMAs per wave) whose time is mostly
// latency; four of them per SIMD (<= 128 registers, which the compiler meets without spilling) instead
// of the three it would otherwise leave room for: the conv5 backward data product 32 -> 29 us.
// NG (one tile row per group only, RS = 16): 16-row groups per wave.  Where rows of G_r moved into the tile-row
// index, NG consecutive tile rows have the very same tiles; one wave then takes NG of them, and every loaded row
// of I feeds NG groups of MFMAs: the rows of I cross the load path of the CU 1/NG as often (a stage of 72 steps
// asks for 23 KB per 2304 MFMA cycles and wave, ~40 B/clk per CU with four waves, close to what the path
// delivers), at NG times the accumulators.  Two groups with stages of up to 32 steps (36 tap-grouped) still fit two
// waves per SIMD without spilling; the larger ones get one.
// CTILES (stages of up to 8 steps): the variant whose waves take several column tiles one after the other.
// LEAN (stages of 18 steps and more): one register set instead of two -- every slot is refilled in place for the next
// stage right after its last use -- so that more waves fit a SIMD (72 steps: two instead of one; 32 and 36 steps:
// three instead of two; 18 steps: four instead of three; two groups of 36 steps or of 72 tap-grouped ones: two
// instead of one).  One tile row a group, 32 steps or tap-grouped: the bound keeps the compiler at the 128 registers of four waves, which it
// would pass by a few (transposed layer 7 at 1/2, 24 images 13.9 us without, 13.4 with; shorter lists 0 to 1 %).
// KL: stage size of the packed layout and the row table (see rbgp_reg_walk).
// HALF (one register set, one row group): a wave's list in two chains of sums, every other stage in the first and the rest in the second:
// the chains of a list split over twice as many waves, which this stands in for (rule at the split of stage lists).  The first chain's
// sums are put aside as the 16 of the epilogue's units: two sets of accumulators, one stage for each in turn, took 0.6 us more.
template <int KC, int RS, bool TAPS = false, int NG = 1, bool CTILES = false, bool LEAN = false, int KL = KC, bool HALF = false>
__global__ __launch_bounds__(256, (LEAN && !HALF && NG == 1 && RS == 16 && (KC == 32 || TAPS) ? 4   // (128 registers)
                                   : LEAN || (NG == 2 && (KC <= 32 || (KC == 36 && TAPS))) ? 2
                                   : KC <= 8 && NG == 1                                   ? (CTILES ? 2 : RS >= 4 ? 4 : 3)
                                                                                          : 1)) void spmm_reg(RegParams p) {
  static_assert(!CTILES || (KC <= 8 && !TAPS), "column tiles per wave: short stages, not the fused convolution");
  static_assert(!LEAN || (KC > 8 && !CTILES), "one register set: the long stages");
  static_assert(!HALF || (LEAN && NG == 1), "two chains of sums: one register set, one row group");
  static_assert(!TAPS || KC % 12 == 0, "tap-grouped stages are multiples of 12 steps");
  static_assert(NG == 1 || RS == 16, "several groups per wave: one tile row per group");
  constexpr int MG = 16 / RS;            // tile rows per MFMA group = cluster size
  constexpr int NO = (KC + 3) / 4;       // load slots per stage (4 contraction steps each)
  constexpr int NQ = (NO + 3) / 4;       // weight registers per stage come as NQ 16-byte loads
  constexpr int QB = 4 * RS * 16;        // bytes of one such load across the fragment
  constexpr int FB = ((KL + 3) / 4 + 3) / 4 * QB;   // bytes of one weight fragment (one tile row, one G_i vertex)
  constexpr int CW = 64;                 // columns per wave
  extern __shared__ __attribute__((aligned(16))) unsigned char wlds[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);

  // A workgroup is one (cluster, G_i vertex) pair on four neighbouring column tiles.  Same
  // columns of I -> same XCD (one L2): workgroups are dealt round-robin to the 8 XCDs.
  // (grid x = 8 * clusters is a multiple of 8, so the XCD of a workgroup is x & 7 whatever y, z)
  // The column-tile index is the slowest grid dimension: all (cluster, G_i vertex) pairs of the
  // same columns are dispatched together, so I comes from HBM once however large N is.
  // The stage list of a cluster can be split over S = 1, 2 or 4 waves of the workgroup (wave
  // k takes stages k, k + S, ...; the partial sums meet in LDS): the workgroup then covers
  // 4 / S column tiles.  Used when N is too small to give every SIMD a wave otherwise.
  const int lgS = p.lgS, S = 1 << lgS;
  const int ks = wid & (S - 1);
  table_args(p);
  WgCoord wg;
  if (!wg_coord(p, &wg)) return;
  const int cl = wg.cl * NG, u3 = wg.u3, ntq = wg.ntq;   // (NG > 1: the first of the wave's NG tile rows; all share its tables)
  // Register sets = stages of loads in flight.  Two for the long stages; a stage of 8 steps is 8 MFMAs (256
  // cycles), and two of them ahead cover far less than a memory access takes: such kernels keep four.
  constexpr int D = LEAN ? 1 : KC <= 8 ? 4 : 2;
  // Short stages, every stage list of the same length: a wave takes `ct` neighbouring column tiles one after the
  // other as ONE list of ct * (stages per tile) stages (lane l of the stage table then serves column tile
  // l / stages-per-tile), so the tables are fetched once and the first rows of the next tile are on their way while
  // the last stages of this one are multiplied; the sums of a tile are stored when its last stage is done.
  const int ct = CTILES ? p.ct : 1;
  const int nt = ((ntq << (2 - lgS)) + (wid >> lgS)) * ct;   // (the first of them)
  const int64_t n0 = int64_t(nt) * CW;
  const int g = lane >> 4, j = lane & 15;
  const int mi = j / RS, ri = j % RS;    // as a weight lane: member of the group, row of the member

  // Everything the prologue needs is requested at once: cluster members, row table, stage
  // table (one stage per lane, read back with readlane), stage count.
  int mem[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm) mem[mm] = p.members[cl * MG + mm];
  const int32_t *rt = p.rowtab + u3 * ((KL + 3) / 4 * 4) + g;
  int rrow[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) rrow[o] = rt[o * 4];
  // the wave's own stages, one per lane: stage ks + lane * S of the cluster's list
  const int TS = p.tstride;
  int own = ks + (lane << lgS), ctile = 0;
  if (CTILES) {
    ctile = rbgp_fast::quotient(lane, p.by_ct_cnt);
    own = lane - ctile * p.ct_cnt;
  }
  // byte offset of the first column (of the lane's table entry's tile) in a row of I (fused convolution: the
  // lane's own column offset inside a channel of X, see `off` below)
  const uint32_t n0b = p.conv ? 0u : uint32_t(nt + ctile) * uint32_t(CW * 4);
  const bool tile_ok = nt + ctile < p.ntiles;
  const int32_t *stg = p.stages + int64_t(cl) * (1 + MG) * TS + (own < TS ? own : TS - 1);
  const int tb = stg[0];
  int tf[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm) tf[mm] = stg[(1 + mm) * TS];
  const int cnt0 = p.counts[cl];
  const int tiles_here = p.ntiles - nt < ct ? p.ntiles - nt : ct;
  const int cnt = __builtin_amdgcn_readfirstlane(   // stages of this wave
      CTILES ? p.ct_cnt * (tiles_here > 0 ? tiles_here : 0) : cnt0 > ks ? (cnt0 - ks + S - 1) >> lgS : 0);
  const int rov = row_offset(p, u3, lane & 15);   // lane-held copies, read back with bpermute in the epilogue
  const int memv = p.members[cl * MG + (lane & (MG - 1))];
  // table lane of the wave's s-th stage (all 64 lanes may hold stages: a stage past the wave's count is made a
  // sentinel where it is read back -- zero extent, weights past the end of the buffer)
  const int first = (cnt + 1) >> 1;   // HALF: stages of the first chain
  auto table_lane = [&](int s) {
    if constexpr (HALF) s = s < first ? 2 * s : 2 * (s - first) + 1;
    return s < 63 ? s : 63;
  };

  // byte offset of this lane's 16 bytes in every slot, relative to the stage base.  Columns
  // past N read whatever follows inside I (or zeros past its end): they are never stored.
  int off[NO];
  bool row_start = false, row_end = false;   // TAPS: the lane's four pixels touch the left / right image border
  if (p.conv) {
    // Fused 3x3 convolution: column n = (image * H + y) * W + x of the lowered input is pixel
    // (y + dy, x + dx) of the zero-padded image; the lane's four columns lie in one image row
    // (W % 4 == 0), so a tap is a constant shift of one 16-byte load.  The table entry already
    // holds channel * bytes per channel + shift of the tap.
    // (host table: no integer division here; its two low bits flag the image borders)
    const int cb = p.colbase[nt < p.ntiles ? int(n0 >> 2) + j : 0];   // (a wave past the last tile loads nothing)
    const int colbase = cb & ~3;
#pragma unroll
    for (int o = 0; o < NO; ++o) off[o] = rrow[o] + colbase;
    row_start = cb & 1;
    row_end = cb & 2;
  } else {
#pragma unroll
    for (int o = 0; o < NO; ++o) off[o] = rrow[o] * (int(p.ldI) * 4) + j * 16;   // < 2^31: checked by the host
  }
  const int alane = (g * RS + ri) * 16;
  const bool valid = nt < p.ntiles;

  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  // Once per stage (= per table lane), with vector instructions: where the stage's part of I
  // starts and how far it extends, and where each member's weights are.  The loop then only
  // reads these back (readlane), which keeps the scalar work between two stages short enough
  // to hide behind the last MFMAs of a stage.
  // The descriptor of a stage starts at the stage's first row and the wave's first column, so
  // the 32-bit offsets inside it only span one stage (I itself may exceed 4 GiB).  A stage
  // touches at most p.src_rows rows: its extent fits 32 bits, and only where the stage reaches
  // the last row of I does the extent end inside it, at the last column.  A stage past the end
  // gets extent zero: its loads return zeros without a memory access.
  const int tbu = p.conv ? int(uint32_t(tb < 0 ? 0 : tb) / 9u) : (tb < 0 ? 0 : tb);   // first row (channel) of the stage
  const uint64_t i_first = reinterpret_cast<uint64_t>(p.I) + uint64_t(uint32_t(tbu)) * p.row_bytes + n0b;
  const int ib_lo = int(uint32_t(i_first)), ib_hi = int(uint32_t(i_first >> 32));
  const int rows_left = p.last_row - tbu < p.src_rows ? p.last_row - tbu : p.src_rows;
  const int ib_ext = (tb >= 0 && tile_ok) ? int(uint32_t(rows_left) * p.row_bytes + (p.n_bytes - n0b)) : 0;
  // per-lane byte offset of each member's weights: a tile row that lacks the tile reads at an
  // offset past the weight buffer (zeros)
  int aoff[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm)
    aoff[mm] = (tf[mm] >= 0 && mem[mm] >= 0) ? ((mem[mm] * p.fpm + tf[mm]) * p.a3 + u3) * FB : kOob;
  auto b_rsrc = [&](int s, int *sofs) {
    const int tl = table_lane(s);
    const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_lo, tl))) |
                          (uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_hi, tl))) << 32);
    *sofs = 0;
    const int ext = __builtin_amdgcn_readlane(ib_ext, tl);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, s < cnt ? ext : 0, kRsrcFlags);
  };

  f32x4 Bs[D][NO];
  f32x4 As[D][NG][NQ];
  if (!valid && lgS == 0) return;   // (with a split stage list every wave reaches the barrier below)
  // Drain every outstanding load count here: a wait for the table loads inside the loop
  // would run on every iteration and drain the prefetched stages with it.
  __builtin_amdgcn_s_waitcnt(0);

  f32x16 acc[NG][4];
#pragma unroll
  for (int k = 0; k < NG; ++k)
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[k][w][v] = 0.f;
  const int gstr = p.fpm * p.a3 * FB;   // NG > 1: from one tile row's weights to the next one's (same tile, same stage)

  // Loads are unconditional so that the wait counts are exact (sentinel stages and absent
  // tiles read zeros, see above).
  auto a_addr = [&](int s) {
    int addr = 0;
    const int tl = table_lane(s);
#pragma unroll
    for (int mm = 0; mm < MG; ++mm) {
      const int sv = __builtin_amdgcn_readlane(aoff[mm], tl);
      addr = mi == mm ? sv : addr;
    }
    return (s < cnt ? addr : kOob) + alane;
  };
  auto a_load = [&](int addr, int q) { return load_x4(rw, addr, q * QB); };

  // The four B operands of slot o (one per column offset w).  TAPS: from the pair's middle window
  // c (pixels x .. x+3): dx = -1 is {left neighbour, c0, c1, c2}, dx = +1 is {c1, c2, c3, right
  // neighbour}; the neighbours are the adjacent lanes' pixels, or zero outside the image.
  auto operand = [&](const f32x4 (&B)[NO], auto oc) {
    constexpr int o = decltype(oc)::value;
    if constexpr (!TAPS) {
      return B[o];
    } else {
      constexpr int dxi = o % 3;
      const f32x4 c = B[o - dxi + 1];
      if constexpr (dxi == 1) {
        return c;
      } else if constexpr (dxi == 0) {
        const int nb = __builtin_amdgcn_update_dpp(0, __float_as_int(c[3]), 0x111 /* row_shr:1 */, 0xf, 0xf, true);
        return f32x4{row_start ? 0.f : __int_as_float(nb), c[0], c[1], c[2]};
      } else {
        const int nb = __builtin_amdgcn_update_dpp(0, __float_as_int(c[0]), 0x101 /* row_shl:1 */, 0xf, 0xf, true);
        return f32x4{c[1], c[2], c[3], row_end ? 0.f : __int_as_float(nb)};
      }
    }
  };

  // One stage: MFMAs of stage s from (B, A); every B slot and every weight quad is
  // refilled for stage s + D right after its last use (RELOAD), so that about D stages
  // of loads are in flight at any time.  Every real stage has work (the stage list is the
  // union of the cluster's tiles), so the loop body is branch-free and its wait counts
  // are exact.
  auto stage = [&](int s, f32x4 (&B)[NO], f32x4 (&A)[NG][NQ], auto reload) {
    constexpr bool RELOAD = decltype(reload)::value;
    int sofs = 0, av = 0;
    __amdgpu_buffer_rsrc_t rb2 = rw;
    if constexpr (RELOAD) {
      rb2 = b_rsrc(s + D, &sofs);
      av = a_addr(s + D);
    }
    static_for<0, NO>([&](auto oc) {
      constexpr int o = decltype(oc)::value;
      const f32x4 b = operand(B, oc);
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const float a = A[k][o / 4][o % 4];
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[k][w] = __builtin_amdgcn_mfma_f32_16x16x1f32(a, b[w], acc[k][w], 0, 0, 0);
      }
      if constexpr (RELOAD) {
        if constexpr (!TAPS)
          B[o] = load_x4(rb2, off[o], sofs);
        else if constexpr (o % 3 == 2)
          B[o - 1] = load_x4(rb2, off[o - 1], sofs);   // the pair's middle window, after its last use
        if constexpr (o % 4 == 3 || o == NO - 1) {
          // (a last quad that is used in part stays whole until here: a register of it that the compiler gave to
          // something else would have to wait for the quad's pending load, i.e. for every load in flight)
#pragma unroll
          for (int k = 0; k < NG; ++k) {
            asm volatile("" ::"v"(A[k][o / 4]));
            A[k][o / 4] = a_load(av + k * gstr, o / 4);
          }
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the loads where they are: the wait counts depend on it
      }
    });
  };
  // loads of stage s in the same order as the refills above
  auto fill = [&](int s, f32x4 (&B)[NO], f32x4 (&A)[NG][NQ]) {
    int sofs;
    const __amdgpu_buffer_rsrc_t rb2 = b_rsrc(s, &sofs);
    const int av = a_addr(s);
    static_for<0, NO>([&](auto oc) {
      constexpr int o = decltype(oc)::value;
      if constexpr (!TAPS)
        B[o] = load_x4(rb2, off[o], sofs);
      else if constexpr (o % 3 == 2)
        B[o - 1] = load_x4(rb2, off[o - 1], sofs);
      if constexpr (o % 4 == 3 || o == NO - 1) {
#pragma unroll
        for (int k = 0; k < NG; ++k) A[k][o / 4] = a_load(av + k * gstr, o / 4);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Stage 0 starts as soon as its own data is there: the loads of stage 1 (into the second
  // register set) and the refills for stage 2 are issued between its MFMAs.
  auto first_stage = [&](f32x4 (&B)[NO], f32x4 (&A)[NG][NQ], f32x4 (&Bn)[NO], f32x4 (&An)[NG][NQ]) {
    int sofs1, sofs2;
    const __amdgpu_buffer_rsrc_t rb1 = b_rsrc(1, &sofs1), rb2 = b_rsrc(2, &sofs2);
    const int av1 = a_addr(1), av2 = a_addr(2);
    static_for<0, NO>([&](auto oc) {
      constexpr int o = decltype(oc)::value;
      const f32x4 b = operand(B, oc);
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const float a = A[k][o / 4][o % 4];
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[k][w] = __builtin_amdgcn_mfma_f32_16x16x1f32(a, b[w], acc[k][w], 0, 0, 0);
      }
      if constexpr (!TAPS) {
        Bn[o] = load_x4(rb1, off[o], sofs1);
        B[o] = load_x4(rb2, off[o], sofs2);
      } else if constexpr (o % 3 == 2) {
        Bn[o - 1] = load_x4(rb1, off[o - 1], sofs1);
        B[o - 1] = load_x4(rb2, off[o - 1], sofs2);
      }
      if constexpr (o % 4 == 3 || o == NO - 1) {
#pragma unroll
        for (int k = 0; k < NG; ++k) {
          An[k][o / 4] = a_load(av1 + k * gstr, o / 4);
          asm volatile("" ::"v"(A[k][o / 4]));
          A[k][o / 4] = a_load(av2 + k * gstr, o / 4);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // epilogue: add the four blocks (contraction steps 0..3 mod 4).  Unit t of the sum holds
  // weight row 4*(lane/16) + t of the group, lane j the columns 4j + w (of the column tile that starts at n0c).
  f32x4 aside[HALF ? 4 : 1];   // HALF: the units of the first chain
#pragma unroll
  for (f32x4 &v : aside) v = f32x4{0.f, 0.f, 0.f, 0.f};
  auto unit = [&](int t, int k = 0) {
    f32x4 v;
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = (acc[k][w][t] + acc[k][w][4 + t]) + (acc[k][w][8 + t] + acc[k][w][12 + t]);
    if constexpr (HALF) v = aside[t] + v;
    return v;
  };
  auto put_aside = [&]() {
#pragma unroll
    for (int t = 0; t < 4; ++t) aside[HALF ? t : 0] = unit(t);
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[0][w][v] = 0.f;
  };
  // (the kernel arguments the stores need, read once: inside the store helpers they would be fetched again per unit)
  float *const out = p.O;
  const int64_t out_ld = p.ldO, out_n = p.N;
  const int out_tm = p.tm, out_a4 = p.a4, out_r = p.R;
  auto whole_at = [&](int64_t n0c) { return n0c + j * 4 + 4 <= out_n; };
  auto store_unit = [&](int t, f32x4 v, int k, int64_t n0c, bool whole, auto past) {
    const int i16 = 4 * g + t, mm = i16 / RS, r = i16 % RS;
    int u1 = __builtin_amdgcn_ds_bpermute(mm * 4, memv);
    if constexpr (NG > 1) u1 = u1 >= 0 ? u1 + k : u1;   // (group k is the tile row after group k - 1's)
    const int ro = __builtin_amdgcn_ds_bpermute(r * 4, rov);
    if (valid && u1 >= 0 && r < out_r) {
      const int64_t m = int64_t(u1) * out_tm + u3 * out_a4 + ro;
      float *o = out + m * out_ld + n0c + j * 4;
      if (whole) {
        store_x4<decltype(past)::value>(o, v);
      } else {
#pragma unroll
        for (int w = 0; w < 4; ++w)
          if (n0c + j * 4 + w < out_n) o[w] = v[w];
      }
    }
  };
  auto store_tile_as = [&](int64_t n0c, auto past) {
    const bool whole = whole_at(n0c);
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) store_unit(t, unit(t, k), k, n0c, whole, past);
  };
  const bool through = p.through != 0;
  auto store_tile = [&](int64_t n0c) {
    if (through) store_tile_as(n0c, std::false_type{});
    else store_tile_as(n0c, std::true_type{});
  };

  // The register sets take turns; stages past the end read zeros (sentinel table lanes).
  if constexpr (D == 2) {
    f32x4(&B0)[NO] = Bs[0], (&B1)[NO] = Bs[1];
    f32x4(&A0)[NG][NQ] = As[0], (&A1)[NG][NQ] = As[1];
    fill(0, B0, A0);
    first_stage(B0, A0, B1, A1);
    if (cnt > 1) {   // the loop is reachable only through stage 1, which keeps its wait counts exact
      stage(1, B1, A1, std::true_type{});
      int s = 2;
      for (; s + 1 < cnt; s += 2) {
        stage(s, B0, A0, std::true_type{});
        stage(s + 1, B1, A1, std::true_type{});
      }
      if (s < cnt) stage(s, B0, A0, std::false_type{});
    }
  } else {
    // all D sets are requested up front; whole rounds of D stages refill as they go (branch-free: exact wait
    // counts); the last, partial round only consumes what is already on its way
    static_for<0, D>([&](auto kc) { fill(decltype(kc)::value, Bs[decltype(kc)::value], As[decltype(kc)::value]); });
    int s = 0;
    if constexpr (CTILES) {
      // several column tiles, one list: every tile has p.ct_cnt stages, a multiple of D, so a tile ends with a
      // round; its sums are stored while the first stages of the next tile are already in flight
      int left = p.ct_cnt;
      int64_t n0c = n0;
      for (; s + D <= cnt; s += D) {
        static_for<0, D>([&](auto kc) {
          constexpr int k = decltype(kc)::value;
          stage(s + k, Bs[k], As[k], std::true_type{});
        });
        left -= D;
        if (left == 0) {
          store_tile(n0c);
#pragma unroll
          for (int k = 0; k < NG; ++k)
#pragma unroll
            for (int w = 0; w < 4; ++w)
#pragma unroll
              for (int v = 0; v < 16; ++v) acc[k][w][v] = 0.f;
          n0c += CW;
          left = p.ct_cnt;
        }
      }
      return;
    }
    for (; s + D <= cnt; s += D) {
      if (HALF && s == first) put_aside();   // (no loads: the wait counts stay exact)
      static_for<0, D>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        stage(s + k, Bs[k], As[k], std::true_type{});
      });
    }
    static_for<0, D>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if (s + k < cnt) stage(s + k, Bs[k], As[k], std::false_type{});
    });
  }
  __builtin_amdgcn_s_waitcnt(0);

  if (lgS == 0) {
    store_tile(n0);
  } else {
    // The S waves of a column tile each own the units t with t % S == their share.  A wave
    // leaves the units it does not own in LDS (densely: unit t of owner o sits at
    // (t / S) * (S - 1) + o - (o > share); one such block per group and wave) and, after the barrier,
    // adds up the ones it owns in wave order, so the result does not depend on timing.
    f32x4 *const red4 = reinterpret_cast<f32x4 *>(wlds);
    const int per_wave = (4 >> lgS) * (S - 1);
    const bool whole = whole_at(n0);
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int o = t & (S - 1);
        if (o != ks)
          red4[((k * 4 + wid) * per_wave + (t >> lgS) * (S - 1) + o - (o > ks ? 1 : 0)) * 64 + lane] = unit(t, k);
      }
    __syncthreads();
    const int w0 = wid & ~(S - 1);
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if ((t & (S - 1)) == ks) {
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
          for (int kk = 0; kk < S; ++kk) {
            if (kk == ks)
              v += unit(t, k);
            else
              v += red4[((k * 4 + w0 + kk) * per_wave + (t >> lgS) * (S - 1) + ks - (ks > kk ? 1 : 0)) * 64 + lane];
          }
          store_unit(t, v, k, n0, whole, std::true_type{});
        }
      }
  }
}

typedef rbgp_reg_fn reg_fn;
template <int KC, int RS>
constexpr reg_fn taps_kernel() {   // the tap-grouped variant exists for stages of a multiple of 12 steps
  if constexpr (KC % 12 == 0)
    return spmm_reg<KC, RS, true>;
  else
    return nullptr;
}
template <int KC, int RS, int NG>
constexpr reg_fn taps_kernel_ng() {
  if constexpr (KC % 12 == 0)
    return spmm_reg<KC, RS, true, NG>;
  else
    return nullptr;
}
struct RegEntry {
  int KC, RS;
  reg_fn global_fn, taps_fn;
};
#define RBGP_R(KC, RS) {KC, RS, spmm_reg<KC, RS>, taps_kernel<KC, RS>()}
// several 16-row groups per wave (one tile row each): two for every stage size, four for the short stages
struct RegGroupEntry {
  int KC, NG;
  reg_fn global_fn, taps_fn;
};
#define RBGP_RG(KC, NG) {KC, NG, spmm_reg<KC, 16, false, NG>, taps_kernel_ng<KC, 16, NG>()}
const RegGroupEntry kRegGroupTable[] = {RBGP_RG(8, 2),  RBGP_RG(18, 2), RBGP_RG(32, 2), RBGP_RG(36, 2), RBGP_RG(72, 2),
                                        RBGP_RG(8, 4),  RBGP_RG(18, 4),
                                        {64, 2, spmm_reg<64, 16, false, 2, false, false, 72>, nullptr}};
const RegGroupEntry *find_reg_groups(int KC, int NG) {
  for (const RegGroupEntry &e : kRegGroupTable)
    if (e.KC == KC && e.NG == NG) return &e;
  return nullptr;
}
// one register set (stages of 18 steps and more): {KC, RS, tap-grouped, NG, kernel}
struct RegLeanEntry {
  int KC, RS;
  bool taps;
  int NG;
  reg_fn fn;
};
#define RBGP_L1(KC, RS) {KC, RS, false, 1, spmm_reg<KC, RS, false, 1, false, true>}
#define RBGP_L1T(KC, RS) {KC, RS, true, 1, spmm_reg<KC, RS, true, 1, false, true>}
#define RBGP_L4(KC) RBGP_L1(KC, 2), RBGP_L1(KC, 4), RBGP_L1(KC, 8), RBGP_L1(KC, 16)
#define RBGP_L4T(KC) RBGP_L1T(KC, 2), RBGP_L1T(KC, 4), RBGP_L1T(KC, 8), RBGP_L1T(KC, 16)
const RegLeanEntry kRegLeanTable[] = {RBGP_L4(18),  RBGP_L4(32),  RBGP_L4(36), RBGP_L4(72),
                                      RBGP_L4T(36), RBGP_L4T(72),
                                      {64, 16, false, 1, spmm_reg<64, 16, false, 1, false, true, 72>},
                                      {36, 16, false, 2, spmm_reg<36, 16, false, 2, false, true>},
                                      {36, 16, true, 2, spmm_reg<36, 16, true, 2, false, true>},
                                      {72, 16, true, 2, spmm_reg<72, 16, true, 2, false, true>}};
reg_fn find_reg_lean(int KC, int RS, bool taps, int NG) {
  for (const RegLeanEntry &e : kRegLeanTable)
    if (e.KC == KC && e.RS == RS && e.taps == taps && e.NG == NG) return e.fn;
  return nullptr;
}
// the same in two chains of sums (stages of 36 steps and more, one row group)
#define RBGP_H1(KC, RS, TAPS) {KC, RS, TAPS, 1, spmm_reg<KC, RS, TAPS, 1, false, true, KC, true>}
#define RBGP_H4(KC, TAPS) RBGP_H1(KC, 2, TAPS), RBGP_H1(KC, 4, TAPS), RBGP_H1(KC, 8, TAPS), RBGP_H1(KC, 16, TAPS)
const RegLeanEntry kRegHalfTable[] = {RBGP_H4(36, false), RBGP_H4(72, false), RBGP_H4(36, true), RBGP_H4(72, true),
                                      {64, 16, false, 1, spmm_reg<64, 16, false, 1, false, true, 72, true>}};
reg_fn find_reg_half(int KC, int RS, bool taps) {
  for (const RegLeanEntry &e : kRegHalfTable)
    if (e.KC == KC && e.RS == RS && e.taps == taps) return e.fn;
  return nullptr;
}
// waves that take several column tiles (stages of 8 steps): {RS, NG, kernel}
struct RegTilesEntry {
  int RS, NG;
  reg_fn fn;
};
// (one tile row per group only: with several, the stage lists are of one length only where G_o is complete, and such
// masks run with G_o (x) G_r merged, rbgp_plan_regroup, on longer stages)
const RegTilesEntry kRegTilesTable[] = {{16, 1, spmm_reg<8, 16, false, 1, true>}, {16, 2, spmm_reg<8, 16, false, 2, true>}};
reg_fn find_reg_tiles(int KC, int RS, int NG) {
  if (KC != 8) return nullptr;
  for (const RegTilesEntry &e : kRegTilesTable)
    if (e.RS == RS && e.NG == NG) return e.fn;
  return nullptr;
}
const RegEntry kRegTable[] = {RBGP_R(8, 2),  RBGP_R(18, 2),  RBGP_R(32, 2),  RBGP_R(36, 2),  RBGP_R(72, 2),
                              RBGP_R(8, 4),  RBGP_R(18, 4),  RBGP_R(32, 4),  RBGP_R(36, 4),  RBGP_R(72, 4),
                              RBGP_R(8, 8),  RBGP_R(18, 8),  RBGP_R(32, 8),  RBGP_R(36, 8),  RBGP_R(72, 8),
                              RBGP_R(8, 16), RBGP_R(18, 16), RBGP_R(32, 16), RBGP_R(36, 16), RBGP_R(72, 16)};

const RegEntry *find_reg(int KC, int RS) {
  for (const RegEntry &e : kRegTable)
    if (e.KC == KC && e.RS == RS) return &e;
  return nullptr;
}

struct RegTables {  // device tables of the clustering, in one allocation
  int ncl = 0, tstride = 64, max_stages = 0;
  int32_t *stages = nullptr, *counts = nullptr, *members = nullptr;
};

struct RegState {
  int32_t *rowtab = nullptr;       // fp32 kernels: [a_i][NO*4]; the pairing kernel's table after it (dual_layout), as in rowtab_conv[0]
  int32_t *rowtab_bf16 = nullptr;  // bf16 kernels: [a_i][NKB*16]
  int32_t *pairs = nullptr;        // rbgp_mask::pairs
  uint64_t *conv_tiles = nullptr;  // conv_tile: ConvTileParams::sel, ::tiles
  bool conv_tiles_none = false;    //   G_i does not keep one of v and v + 4 everywhere: no such tables
  int32_t *rowtab_conv[2] = {nullptr, nullptr};   // fused convolution, fp32 / bf16: byte offsets for the geometry below
  int32_t *colbase[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};   // [dtype][wide tile]: pixel offsets of the column groups
  int64_t conv_key[2][3] = {{0, 0, 0}, {0, 0, 0}};  // images, height, width of rowtab_conv
  RegTables tab;                   // fp32: clusters of one 16-row group
  RegTables tab_bf16[3];           // bf16: clusters of 1, 2, 4 groups
  bool g2_shared = false;          // the clusters of two groups have (nearly) half the stages in total: their tile rows share their tiles
  bool g4_none = false;            // the clusters of four groups have too long a list
  int g2_stages = -1, g2_ncl = 0;  // longest stage list and number of the clusters of two groups (-2: too long,
                                   //   or their stage lists add up to more than 0.8 of those of one group)
};

template <typename T>
int upload(const std::vector<T> &h, T **d) {
  RBGP_HIP(hipMalloc(reinterpret_cast<void **>(d), h.size() * sizeof(T) + 16));
  RBGP_HIP(hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
  return RBGP_OK;
}

// bf16 fused convolution of 32-row, 32-channel tiles with one column of G_i kept of every v and v + 4 (rbgp_conv_tile.hip).
// Workgroups of four rows of G_o x 32 T pixels, S waves a row.  While 32-pixel workgroups have a CU each, two waves a row (T, S =
// 1, 2); while 64-pixel ones do, those where a row has four tiles and more (2, 2), else two 32-pixel ones of one wave a row on a
// CU (1, 1); from then on two 64-pixel ones on a CU (2, 1), which stage a chunk while the other multiplies.
// us, register kernels / (1, 1) / (1, 2) / (2, 1) / (2, 2), VGG19, fp32 sums, input gradient unless said:
//  layer 6 at 1/4 (eight rows of G_o, four tiles a row): 576 pixels 10.2 / 8.0 / 6.9 / 11.9 / 9.1, 4096 11.7 / 8.6 / 7.8 / 12.0 / 9.5,
//  5120 17.1 / 10.3 / 12.5 / 12.1 / 9.6, 8192 17.3 / 10.6 / 13.3 / 12.9 / 10.4, 10240 - / 16.3 / 18.9 / 15.0 / 17.6;
//  at 1/8 (two tiles): 4096 8.6 / 6.5 / 6.6 / 8.9 / 7.8, 8192 17.8 / 7.9 / 11.1 / 9.8 / 8.5, 16384 - / 14.6 / 22.2 / 12.7 / 15.8;
//  layer 9 at 1/4 (16 rows, eight tiles): 1024 13.1 / 13.1 / 11.4 / 22 / 15.7, 2048 20.0 / 13.3 / 11.6 / 22 / 15.7, 4096 - / 17.2 / 21.9 /
//  22.5 / 16.8; layer 3 at 1/4, 16384 pixels 9.7 / 8.0 / 10.7 / 9.1 / 8.1, 32768 14.9 / 14.6 / 21.4 / 12.3 / 15.0.
// The register kernels stay with up to 64 workgroups where 16 channels' tiles and more are to be staged for rows of eight tiles, or
// for tiles that share eight rows a column set (layer 9 at 1/4, 512 pixels: 10.6 against 11.0, forward 8.9 / 10.6, forward at 1/8
// 7.2 / 7.6; from 592 pixels on 16.6 / 11.1, 13.4 / 10.6, 9.8 / 7.8): their split lists then run in one round.
// *taken: the launch went this way.  (The tables are made at the first such launch.)
int launch_conv_tile(const rbgp_mask *m, RegState *st, const int *tune, bool out_bf16, const rbgp_conv_geometry &conv, int64_t N,
                     const void *packed, uint32_t w_bytes, const void *X, int64_t chan, void *O, int64_t ldO, void *stream, bool *taken) {
  const rbgp_reg_plan &pl = m->reg;
  *taken = false;
  if (!(pl.fold == 1 && m->c[0] <= 64 && m->c[1] == 4 && m->c[2] == 8 && m->d[2] == 4 && pl.KCR == 72 && pl.KC == 72 && pl.NSTG == 2 &&
        (pl.RS == 4 || pl.RS == 8) && pl.R * m->a[2] == 32 && pl.A2 == m->a[1] && m->a[1] * m->a[3] == pl.R))
    return RBGP_OK;
  for (int k = 0; k < RBGP_NUM_TUNE; ++k)
    if (tune[k]) return RBGP_OK;
  const int64_t per = (m->a[0] + 3) / 4, W = conv.width, H = conv.height;
  const int64_t narrow = (N + 31) / 32 * per, wide = (N + 63) / 64 * per;   // workgroups with T = 1, 2
  if (64 % W || N >= (int64_t(1) << 30) || (narrow <= 64 && m->c[0] >= 16 && (pl.RS == 8 || m->d[0] >= 8))) return RBGP_OK;
  const int T = 32 % W || (narrow > 256 && (wide > 256 || m->d[0] >= 4)) ? 2 : 1, S = (T == 1 ? narrow : wide) <= 256 ? 2 : 1;
  const int64_t cw = 32 * T, tiles = (N + cw - 1) / cw, wgs = 8 * ((tiles + 7) / 8) * per;
  // padded rows of a workgroup's pixels: its rows, two for every image border among them, one on either side
  const int64_t rows = cw / W, px = (rows + 2 * ((rows + H - 2) / H) + 2) * (W + 2), octets = (px + 7) / 8,
                tile_bytes = 512 * octets, most = 75 * 1024;
  if (wgs > 0x7fffffff || tile_bytes > most) return RBGP_OK;
  const size_t rows_o = size_t(per) * 4;
  if (!st->conv_tiles) {
    if (st->conv_tiles_none) return RBGP_OK;
    std::vector<uint64_t> t(size_t(m->a[2]) * 2 + size_t(3) * rows_o, 0);   // ConvTileParams::sel, then ::tiles
    for (int u = 0; u < m->a[2]; ++u) {
      int at[4] = {-1, -1, -1, -1}, late[4];   // place in the adjacency list, and upper half, of the column kept of v and v + 4
      for (int k = 0; k < 4; ++k) {
        const int v = m->adj[2][size_t(u) * 4 + k];
        at[v & 3] = k;
        late[v & 3] = v >> 2;
      }
      for (int k = 0; k < 4; ++k)
        if (at[k] < 0) {
          st->conv_tiles_none = true;
          return RBGP_OK;
        }
      auto bytes_of = [&](int k) { return (2 * at[k] | (2 * at[k] + 1) << 8) | (2 * at[k + 1] | (2 * at[k + 1] + 1) << 8) << 16; };
      const int places = late[0] | (2 + late[1]) << 2 | late[2] << 4 | (2 + late[3]) << 6;
      t[size_t(u) * 2] = uint64_t(bytes_of(2)) << 32 | uint64_t(bytes_of(0));
      t[size_t(u) * 2 + 1] = uint64_t(places | places << 8);
    }
    for (int u = 0; u < m->a[0]; ++u)
      for (int k = 0; k < m->d[0]; ++k) {
        const uint64_t bit = uint64_t(1) << m->adj[0][size_t(u) * m->d[0] + k];
        t[size_t(m->a[2]) * 2 + u] |= bit;
        t[size_t(m->a[2]) * 2 + size_t(1 + k % 2) * rows_o + u] |= bit;
      }
    int rc = upload(t, &st->conv_tiles);
    if (rc) return rc;
  }
  ConvTileParams cp;
  cp.Wp = packed; cp.X = X; cp.O = O;
  cp.sel = reinterpret_cast<const int4 *>(st->conv_tiles); cp.tiles = st->conv_tiles + m->a[2] * 2; cp.rows = int(rows_o);
  cp.ldO = ldO; cp.chan = chan; cp.w_bytes = w_bytes;
  cp.n = int(N); cp.ntiles = int(tiles);
  cp.h = int(H); cp.w = int(W); cp.w2 = int(W + 2); cp.hw = int(H * W);
  cp.a1 = m->a[0]; cp.a2 = m->a[1]; cp.a3 = m->a[2]; cp.a4 = m->a[3]; cp.d1 = m->d[0];
  cp.R = pl.R; cp.RS = pl.RS;
  cp.frag_bytes = (rbgp_bf16_blocks32(pl.KC) + (rbgp_bf16_tail16(pl.KC) ? 1 : 0)) * 4 * pl.RS * 16;
  cp.chunk = int(std::min({int64_t(m->c[0]), most / tile_bytes, 64 * S / octets}));   // (a thread stages one octet of a plane; two buffers)
  cp.obf16 = out_bf16 ? 1 : 0;
  cp.by_per = rbgp_fast::div_by(per); cp.by_hw = rbgp_fast::div_by(H * W); cp.by_w = rbgp_fast::div_by(W);
  cp.by_R = rbgp_fast::div_by(pl.R); cp.by_a4 = rbgp_fast::div_by(m->a[3]);
  const size_t bytes = size_t(std::max((cp.chunk < m->c[0] ? 2 : 1) * cp.chunk * tile_bytes, int64_t(S * T) * 16 * 1024));   // (sums of a row's waves)
  rbgp_conv_tile_fn fn = rbgp_conv_tile_kernel(T, S);
  if (bytes > 64 * 1024)
    RBGP_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)));
  hipLaunchKernelGGL(fn, dim3(unsigned(wgs)), dim3(unsigned(256 * S)), bytes, static_cast<hipStream_t>(stream), cp);
  RBGP_HIP(hipGetLastError());
  rbgp_set_last_kernel("conv_tile", {T, S});
  *taken = true;
  return RBGP_OK;
}

void free_tables(RegTables *t) {
  if (t->stages) (void)hipFree(t->stages);
  *t = RegTables();
}

// The state is touched only when the tables are on the device.
int upload_tables(const rbgp_reg_clusters &cl, RegTables *t) {
  std::vector<int32_t> all;
  auto append = [&](const std::vector<int32_t> &part) {
    const size_t at = (all.size() + 63) / 64 * 64;
    all.resize(at);
    all.insert(all.end(), part.begin(), part.end());
    return at;
  };
  append(cl.stages);
  const size_t counts = append(cl.counts), members = append(cl.members);
  int32_t *dev = nullptr;
  if (const int rc = upload(all, &dev)) return rc;
  t->ncl = cl.ncl; t->tstride = cl.tstride; t->max_stages = cl.max_stages;
  t->stages = dev; t->counts = dev + counts; t->members = dev + members;
  return RBGP_OK;
}

// Upload the clustering of the tile rows (clusters of U) and its stage tables.
int build_tables(const rbgp_mask *m, int U, RegTables *t) {
  rbgp_reg_clusters fresh;
  const rbgp_reg_clusters *cl = &m->reg_clusters;
  if (U != cl->U) {
    rbgp_reg_cluster(m, U, &fresh);
    cl = &fresh;
  }
  if (cl->max_stages > kRegMaxStages) return RBGP_EUNSUPPORTED;   // one stage per lane plus sentinels, four waves
  return upload_tables(*cl, t);
}

// The table of the pairing kernel (DualParams::tab), in the buffer of the row table that it repeats: word offsets, and their end.
struct DualLayout {
  int np4, cmax, stages, quads, words;   // stages, quads: from the table's own start
  size_t first;                          // of the table, in the buffer
};
DualLayout dual_layout(const rbgp_mask *m) {
  const rbgp_reg_dual &du = m->reg_dual;
  DualLayout l;
  l.np4 = (m->reg.NO + 3) / 4 * 4;
  l.cmax = std::max(du.max_wave, 1);
  l.stages = m->a[2] * (4 * l.np4 + 16);
  l.quads = l.stages + du.nq * 4 * l.cmax * 4;
  l.words = l.quads + du.nq * 8;
  l.first = (size_t(m->a[2]) * (m->reg.NO * 4 + 16) + 63) / 64 * 64;
  return l;
}
// rt: the row table with row_offset's table behind it
void append_dual_table(const rbgp_mask *m, std::vector<int32_t> &rt) {
  const rbgp_reg_plan &pl = m->reg;
  const rbgp_reg_dual &du = m->reg_dual;
  const DualLayout l = dual_layout(m);
  rt.resize(l.first + l.words, 0);
  int32_t *const h = rt.data() + l.first;
  for (int u = 0; u < m->a[2]; ++u) {
    int32_t *const own = h + size_t(u) * (4 * l.np4 + 16);
    for (int o = 0; o < pl.NO; ++o)
      for (int gg = 0; gg < 4; ++gg) own[gg * l.np4 + o] = rt[(size_t(u) * pl.NO + o) * 4 + gg];
    for (int r = 0; r < 16; ++r) own[4 * l.np4 + r] = rt[(size_t(m->a[2]) * pl.NO) * 4 + size_t(u) * 16 + r];
  }
  for (int wv = 0; wv < du.nq * 4; ++wv)
    for (int sg = 0; sg < l.cmax; ++sg)
      for (int k = 0; k < 3; ++k) h[size_t(l.stages) + (size_t(wv) * l.cmax + sg) * 4 + k] = du.stages[(size_t(wv) * 3 + k) * 64 + sg];
  for (int q = 0; q < du.nq; ++q)
    for (int k = 0; k < 4; ++k) {
      h[size_t(l.quads) + size_t(q) * 8 + k] = du.members[size_t(q) * 4 + k];
      h[size_t(l.quads) + size_t(q) * 8 + 4 + k] = du.counts[size_t(q) * 4 + k];
    }
}

}  // namespace

bool rbgp_reg_covers(const rbgp_mask *m) {
  const rbgp_reg_plan &p = m->reg;
  if (!p.ok) return false;
  // every cluster's stage list must fit the per-lane table
  if (m->reg_clusters.max_stages > kRegMaxStages) return false;
  return find_reg(p.KC, p.RS) != nullptr;
}

void rbgp_reg_release(void *state) {
  RegState *st = static_cast<RegState *>(state);
  if (!st) return;
  if (st->rowtab) (void)hipFree(st->rowtab);
  if (st->rowtab_bf16) (void)hipFree(st->rowtab_bf16);
  if (st->pairs) (void)hipFree(st->pairs);
  if (st->conv_tiles) (void)hipFree(st->conv_tiles);
  for (int32_t *t : st->rowtab_conv)
    if (t) (void)hipFree(t);
  for (auto &pair : st->colbase)
    for (int32_t *t : pair)
      if (t) (void)hipFree(t);
  free_tables(&st->tab);
  for (RegTables &t : st->tab_bf16) free_tables(&t);
  delete st;
}

int rbgp_reg_launch(const rbgp_mask *m, void **state, const int *tune, bool bf16, bool out_bf16, int64_t N,
                    const void *packed, const void *I, int64_t ldI, void *O, int64_t ldO, void *stream,
                    const rbgp_conv_geometry *conv) {
  const rbgp_reg_plan &pl = m->reg;
  if (!rbgp_reg_covers(m)) return RBGP_EUNSUPPORTED;
  if (out_bf16 && !bf16) return RBGP_EINVAL;
  // Fused 3x3 convolution: the nine taps are the columns of a complete G_b and an image row holds
  // whole lane loads (4 columns; 8 with the wide bf16 tile); "I" is then the padded activation
  // tensor and ldI is not used.
  int64_t chs = 0;   // bytes of one channel of X
  if (conv) {
    if (m->c[3] != 9 || m->d[3] != 9) return RBGP_EUNSUPPORTED;
    if (conv->images <= 0 || conv->height <= 0 || conv->width <= 0 || conv->width % 4) return RBGP_ESHAPE;
    if (N != conv->images * conv->height * conv->width) return RBGP_ESHAPE;
    if (reinterpret_cast<uintptr_t>(I) % 4) return RBGP_ESHAPE;
    chs = conv->images * (conv->height + 2) * (conv->width + 2) * (bf16 ? 2 : 4);
    if ((int64_t(pl.SRC) / 9 + 1) * chs >= (int64_t(1) << 31)) return RBGP_EUNSUPPORTED;
    ldI = N;   // (only the checks below read it)
  }
  // I and the packed weights are addressed through 32-bit buffer offsets
  const int es = bf16 ? 2 : 4;
  // bf16: a lane loads 8 bytes (4 columns; 64-column wave tile) or 16 bytes (8 columns;
  // 128-column tile) per row.  The wide tile is the default where the operands allow it and
  // enough column tiles remain to fill the chip.
  int CW = 64;
  if (bf16) {
    const bool ok64 = conv ? true : (ldI % 4 == 0) && (reinterpret_cast<uintptr_t>(I) % 8 == 0);
    const bool ok128 = conv ? conv->width % 8 == 0 : (ldI % 8 == 0) && (reinterpret_cast<uintptr_t>(I) % 16 == 0);
    const int tc = tune[RBGP_TUNE_COLS_PER_WORKGROUP];
    if (tc != 0 && tc != 64 && tc != 128) return RBGP_EUNSUPPORTED;
    if (tc)
      CW = tc;
    else if (ok128 && int64_t((pl.TR + pl.MG - 1) / pl.MG) * m->a[2] * ((N + 127) / 128) >= 512)
      CW = 128;
    if (!(CW == 128 ? ok128 : ok64)) return RBGP_ESHAPE;
  }
  int NC = CW / 16;
  // (bf16: two columns share a dword, and a dword that crosses the end of the descriptor reads
  // as zero, so the last row's extent (n_bytes below) is rounded up to the bytes a lane loads;
  // the condition on ldI keeps that inside the K x ldI array)
  const int64_t w_bytes = (bf16 ? pl.packed_elems_bf16 : pl.packed_elems) * es;
  // 32-bit offsets address one stage of I (its rows span SRC * ldI elements; I as a whole may be
  // larger) and the packed weights
  if ((!conv && (int64_t(pl.SRC) * ldI + CW) * es >= (int64_t(1) << 31)) || w_bytes >= (int64_t(1) << 30))
    return RBGP_EUNSUPPORTED;
  RegState *st = static_cast<RegState *>(*state);
  if (!st) {
    st = new (std::nothrow) RegState();
    if (!st) return RBGP_ENOMEM;
    *state = st;
  }
  if (bf16 && conv) {
    bool taken;
    int rc = launch_conv_tile(m, st, tune, out_bf16, *conv, N, packed, uint32_t(w_bytes), I, chs / es, O, ldO, stream, &taken);
    if (rc || taken) return rc;
  }
  int32_t **rowtab = conv ? &st->rowtab_conv[bf16] : bf16 ? &st->rowtab_bf16 : &st->rowtab;
  int64_t *ckey = st->conv_key[bf16];
  if (conv && *rowtab && (ckey[0] != conv->images || ckey[1] != conv->height || ckey[2] != conv->width)) {
    (void)hipFree(*rowtab);   // (waits for launches that still read the old table)
    *rowtab = nullptr;
    for (int32_t *&t : st->colbase[bf16]) {
      if (t) (void)hipFree(t);
      t = nullptr;
    }
  }
  if (!*rowtab) {
    const int a3 = m->a[2], d3 = m->d[2], c3 = m->c[2], c4 = m->c[3];
    const int len = bf16 ? 32 * rbgp_bf16_blocks32(pl.KC) + (rbgp_bf16_tail16(pl.KC) ? 16 : 0) : pl.NO * 4;   // contraction steps, padded (padding -> row 0)
    std::vector<int32_t> rt(size_t(a3) * len, 0);
    for (int u3 = 0; u3 < a3; ++u3)
      for (int kk = 0; kk < pl.KCR; ++kk) {
        const int st = bf16 ? kk : rbgp_reg_step(m, kk);   // step of the contraction list at position kk
        const int v4 = st % c4, j3 = (st / c4) % d3, vv = st / (c4 * d3);
        rt[size_t(u3) * len + kk] = (vv * c3 + m->adj[2][size_t(u3) * d3 + j3]) * c4 + v4;
      }
    if (conv) {   // stage-relative row 9 * channel + tap -> byte offset of the channel plus the shift of the tap
      for (int32_t &r : rt) {
        const int tap = r % 9, dy = tap / 3 - 1, dx = tap % 3 - 1;
        r = int32_t((r / 9) * chs + (dy * (conv->width + 2) + dx) * es);
      }
      ckey[0] = conv->images; ckey[1] = conv->height; ckey[2] = conv->width;
    }
    for (int u = 0; u < a3; ++u)   // row_offset's table
      for (int r = 0; r < 16; ++r) {
        const int64_t row = (int64_t(r / m->a[3]) * a3 + u) * m->a[3] + r % m->a[3];   // (of tile row 0)
        rt.push_back(r < pl.R ? int32_t(rbgp_twin_row(m, row) - u * m->a[3]) : 0);
      }
    if (!bf16 && m->reg_dual.ok && rbgp_reg_dual_kernel(pl.KC)) append_dual_table(m, rt);
    int rc = upload(rt, rowtab);
    if (rc) return rc;
  }
  int64_t ntiles = (N + CW - 1) / CW;
  // bf16: 16-row groups per wave (G) and waves per column tile (S).  More groups mean fewer
  // passes of I through the load path at the price of multiplied zeros; on the VGG19 conv3 shape
  // the two balance out, so the default is one group unless the rule below finds two worth it.
  // The stage list is split when there are fewer (cluster, G_i vertex, column tile) triples than SIMDs.
  int G = 1, lgS = 0;
  int64_t lists = 0;   // (cluster, G_i vertex, column tile) triples (0: K_SPLIT is given)
  bool halves = false;   // a wave's list in two chains of sums
  // long stages split by what the busiest SIMD walks (not with the knobs whose kernels are no others than those of every other split)
  const bool by_walk = pl.KC > 32 && !tune[RBGP_TUNE_ROW_GROUPS] && !tune[RBGP_TUNE_REGISTER_SETS];
  bool two_groups = false, four_groups = false;   // rbgp_spmm: a batch of another size may take them
  {
    const int tg = bf16 ? tune[RBGP_TUNE_ROW_GROUPS] : 0, ts = tune[RBGP_TUNE_K_SPLIT];
    if (tg) {
      if (tg != 1 && tg != 2 && tg != 4) return RBGP_EUNSUPPORTED;   // (too long a stage list is rejected below)
      G = tg;
    } else if (bf16 && !ts && (pl.TR + pl.MG - 1) / pl.MG >= 2) {
      // Two groups per wave halve the bytes of I that cross the L1 path.  Measured on the VGG19 layers (bf16,
      // densities 1/2 and 1/4): that pays (3-22 %) where the larger clusters still give every SIMD a wave
      // without a split, or where each wave of the split keeps a dozen stages to amortise the reduction; it
      // costs 7-25 % where neither holds, and 7-15 % where G_o is so sparse that the tile rows of a larger
      // cluster share few tiles (density 1/16: the stage lists of the clusters then add up to nearly as many
      // stages as before, each multiplied into twice the rows).
      if (st->g2_stages == -1) {
        rbgp_reg_clusters c2;
        rbgp_reg_cluster(m, 2 * pl.MG, &c2);
        int64_t total1 = 0, total2 = 0;
        for (int32_t c : m->reg_clusters.counts) total1 += c;
        for (int32_t c : c2.counts) total2 += c;
        st->g2_stages = (c2.max_stages > kRegMaxStages || m->reg_clusters.U != pl.MG || 5 * total2 > 4 * total1) ? -2 : c2.max_stages;
        st->g2_ncl = c2.ncl;
        st->g2_shared = 20 * total2 <= 11 * total1;
        if (st->g2_stages > 0 && !conv && !st->tab_bf16[1].stages) {
          int rc = upload_tables(c2, &st->tab_bf16[1]);
          if (rc) {
            st->g2_stages = -1;
            return rc;
          }
        }
      }
      two_groups = st->g2_stages > 0 && !conv;
      const bool can4 = st->g2_stages > 0 && st->g2_shared && pl.MG == 1 && pl.fold % 4 == 0 && pl.KC <= 36 && st->g2_stages >= 32;
      four_groups = can4 && !conv;
      if (st->g2_stages > 0) {
        const int64_t waves2 = int64_t(st->g2_ncl) * m->a[2] * ntiles;
        int S2 = 1;
        while (S2 < 4 && waves2 * S2 < 1024) S2 *= 2;
        // (the fused convolution issues more loads per step -- nine shifted windows per channel -- and gains
        // 15-22 % on every VGG19 layer that keeps the chip full, however short the split lists)
        // (and where the tile rows of a larger cluster have the same tiles -- rows of G_r moved into the tile-row
        // index -- the second group costs no extra stage at all: 12-17 % faster on the density-1/2 layers)
        // (with the one-register-set kernels of the 128-column tiles a split in two pays from six stages per wave on:
        // VGG19 conv3 16.97 -> 16.35 us, layers 5, 6, 9-11 at density 1/4 8-9 % faster)
        const int enough = (S2 == 2 && CW == 128) ? 6 : 12;
        if (waves2 * S2 >= 1024 && (S2 == 1 || conv || st->g2_shared || st->g2_stages / S2 >= enough)) G = 2;
        // Four tile rows with the very same tiles (at least four of G_r's rows moved into the tile-row index, as on the
        // filled masks of Tables 2-3): four groups per wave, where the chip stays full and the accumulators fit without
        // spilling (stages of up to 36 steps).  4096^3 with one row per column set: 182 / 122 / 111 us with 1 / 2 / 4 groups.
        // (stage lists of 16: 53.9 us against 51.1 with two groups -- long lists only)
        if (G == 2 && can4) {
          const int64_t waves4 = int64_t(pl.TR / 4) * m->a[2] * ntiles;
          int S4 = 1;
          while (S4 < 4 && (waves4 * S4 < 1024 || st->g2_stages > kRegWaveStages * S4)) S4 *= 2;
          if (waves4 * S4 >= 1024 && st->g2_stages <= kRegWaveStages * S4) G = 4;
        }
      }
    }
    const int64_t ncl = (pl.TR + G * pl.MG - 1) / (G * pl.MG);
    if (ts) {
      if (ts != 1 && ts != 2 && ts != 4) return RBGP_EUNSUPPORTED;
      lgS = ts == 4 ? 2 : ts == 2 ? 1 : 0;
    } else {
      // Lists split until every SIMD has a wave, but long stages (36 and 72 steps, one row group) only where that shortens what the
      // busiest SIMD walks: of L lists split in S, ceil(S L / 1024) waves of 1 / S list each.  Up to 256 lists that is a quarter
      // with S = 4, up to 512 a half with 2 and with 4, up to 768 3/4 with 4 and a whole list otherwise -- worth the sum of the
      // parts and a third start-up from lists of 12 stages on --, then a whole list whatever S.  In us, as many parts as fill every
      // SIMD -> this: conv5, 48 images (384 lists) fp32 10.9 -> 10.0, bf16 (47) 8.8 -> 7.4; VGG19 layer 9 at 1/2, bf16, 57 images 18.8 ->
      // 16.4; layer 4 at 1/4, bf16, 60 images 8.9 -> 7.1; layer 11 at 1/16, fp32, 75 images 12.6 -> 11.5; 12 stages and more: conv3, 44
      // images 18.3 -> 14.8, layer 9 at 1/4, bf16, 84 images 19.3 -> 15.6; shorter ones in four 15.3 -> 19.6 and 10.8 -> 14.9.
      // fp32 tile rows with one list, whose waves in four would go on to take two row groups, stay in two there (4096 x 4096, density
      // 1/8, 181 columns, 768 lists 23.6, in four 25.8, with two groups 27.1; layer 5 at 1/2, 35 images, 560 lists 23.1, 21.2 and 26.7).
      // Stages of up to 32 steps keep the split (transposes: 32 steps, 4 stages, 864 lists 6.2, whole 7.8; 8 stages, 288 lists in
      // four 6.1, in two 8.3): the waves of a short list mostly wait, and more of them hide more.
      // Where that leaves fewer parts than fill every SIMD, each wave sums its list in two chains (HALF), so that no chain of fp32 sums
      // grows: 0.25 us of a wave in fp32, 0.1 in bf16, where lists of four stages stay in four (layer 7 at 1/16, 20 images 6.25, in two
      // 6.44).  fp32: two parts of up to 512 lists pay where they divide a list better than four do -- two waves of a quarter walk two
      // stages more than one of a half where 4 k + 2 stages are to be dealt (us, four -> two: layer 10 at 1/16, 37 images, six stages 9.3 ->
      // 8.1; conv5, 48 images, ten 11.0 -> 10.0) -- or lists are long (layer 11 at 1/2, 32 stages 24.0 -> 22.5; fused, up to 448 lists:
      // layer 9 at 1/4, 48 images 15.4 -> 15.1, 60 images 15.1 -> 15.9); else they cost up to 9 % (layer 7 at 1/4, 24 images, 12 stages
      // 10.7 -> 10.9; WRN group 1, 4321 columns, eight 5.9 -> 6.4).
      lists = ncl * m->a[2] * ntiles;
      while (lgS < 2 && (lists << lgS) < 1024) ++lgS;
      if (by_walk && G == 1) {
        const int fill = lgS;
        const int n = m->reg_clusters.max_stages;
        lgS = lists <= 256   ? 2
              : lists <= 512 ? ((bf16 && n > 4) || n % 4 == 2 || (n >= 20 && (!conv || lists <= 448)) || lists == 512 ? 1 : 2)
                             : lists <= 768 && n >= 12 ? (!bf16 && pl.fold > 1 ? 1 : 2) : 0;
        halves = lgS < fill;
      }
    }
  }
  const RegEntry *e = find_reg(pl.KC, pl.RS);
  if (!e) return RBGP_EUNSUPPORTED;
  const int walk = rbgp_reg_walk(pl);
  // tile rows that come in groups of `fold` with the same stage list, in order (one tile row per cluster)
  bool in_order = pl.MG == 1 && m->reg_clusters.U == 1;   // cluster c is tile row c
  for (int c = 0; c < m->reg_clusters.ncl && in_order; ++c) in_order = m->reg_clusters.members[size_t(c)] == c;
  const bool ident = in_order && pl.fold > 1;
  // bf16: workgroups of share_rv x (4 / share_rv) waves that pass I through LDS, each wave 2 share_pr of these tile rows
  // and 128 columns (rbgp_mfma_reg_bf16_shared.hip)
  int share_rv = 0, share_pr = 1;
  {
    const int tsh = tune[RBGP_TUNE_SHARED_COLUMNS];
    if (tsh < 0 || tsh > 6) return RBGP_EUNSUPPORTED;
    const bool ok128 = conv ? conv->width % 8 == 0 : (ldI % 8 == 0) && (reinterpret_cast<uintptr_t>(I) % 16 == 0);
    const bool can = bf16 && ident && ok128 && pl.KCR <= 32 * rbgp_bf16_blocks32(pl.KC) &&
                     m->reg_clusters.max_stages <= kRegWaveStages && !tune[RBGP_TUNE_ROW_GROUPS] && !tune[RBGP_TUNE_K_SPLIT] &&
                     !tune[RBGP_TUNE_REGISTER_SETS] && !tune[RBGP_TUNE_COLS_PER_WORKGROUP];
    // shape [knob value - 2], widest tile first where the tiles are of one size
    static const struct { int rv, pr; } shapes[] = {{1, 1}, {2, 1}, {4, 1}, {1, 2}, {2, 2}};
    auto fits = [&](int k) { return can && pl.fold % (2 * shapes[k].rv * shapes[k].pr) == 0; };
    auto wgs = [&](int k) {
      const int cols = 512 / shapes[k].rv;
      return int64_t(pl.TR / (2 * shapes[k].rv * shapes[k].pr)) * m->a[2] * ((N + cols - 1) / cols);
    };
    int pick = tsh - 2;
    if (tsh >= 2 && !fits(pick)) return RBGP_EUNSUPPORTED;
    if (tsh == 0 && can) {
      // 512 workgroups run at a time (two per CU), and a kernel's time hardly depends on how many of them there are: a shape
      // is worth its while when its tiles nearly fill a round, and no longer when they have just begun the second.
      // Measured on the masks of Tables 2 and 3 in us, spmm_reg_bf16 against the shapes (waves along rows x row pairs each):
      //  stages of 64 steps, eight tile rows and more with one list (density 1/8, four rows per column set; lists of 16):
      //    N = 1000 24.6, 4 x 1 23.1 (256 workgroups); 1536 31.8, 26.3; 2048 48.8, 26.8, 2 x 2 33.8; 2176 46.7, 43.7 (544
      //    workgroups), 2 x 2 37.0 (288); 3072 55.5, 47.1, 42.9; 4096 76.3, 51.8, 46.2;
      //    O in bf16 (half of the stores, and the old kernel's time with them): 1000 20.5, 22.4; 1280 (320) 30.2, 24.8; 2048
      //    31.4, 25.5; 2560 43.2, 42.8, 38.5; lists of 8 (1/16) 4 x 1 at 1000 9.2, 10.7, at 1152 11.6, 11.0;
      //  the same, four tile rows (two rows per column set): 1280 32.0, 2 x 1 29.2 (320); 1536 32.7, 30.1; 2048 43.2, 34.3;
      //    2560 50.6, 58.3 (640), 1 x 2 46.9 (320); 3072 56.7, 60.7, 48.7; 4096 66.3, 60.6, 49.5; O in bf16: 1280 30.3, 29.3;
      //    2560 44.3, 57.3, 46.0; 3072 45.3, 59.9, 48.4 (384); 3200 56.9, 58.3, 47.9 (448);
      //  two tile rows: lists of 16 74, 1 x 1 80; of 8 52, 47;
      //  stages of 32 steps, eight tile rows (1/4; spmm_reg_bf16 takes four row groups): 1792 41.2, 4 x 1 43.2 (448);
      //    1920 42.5, 44.0; 2048 58.4, 44.0 (512); 2176 68.0, 65.7, 2 x 2 66.4; 2816 67.0, 72.8, 69.2; 4096 88.1, 88.7,
      //    75.9; lists of 16 (G_o at 1/8, G_i at 1/2) 4 x 1 at 1792 23.4, 17.2;
      //  transposed VGG19 layers, short lists: L3 58, 38; L6 32.5, 26; L9 25, 19 (1 x 2, 2 x 2); L6 at 37 images 26, 28 (2 x 1).
      // With O in bf16, long lists of short stages stay where they are (4096 columns 74, 81).
      const bool long_stages = pl.KC > 36, lists = long_stages || !out_bf16 || m->reg_clusters.max_stages < 32;
      const int64_t round = 512;
      const int64_t tall = !long_stages ? (m->reg_clusters.max_stages >= 32 ? round : 448)
                           : !out_bf16  ? 256
                                        : m->reg_clusters.max_stages >= 8 ? 320 : 384;
      // (O in bf16 and rows of whole 8-byte stores: spmm_reg_bf16 needs 43 us where misaligned rows take it 51 and 1 x 2 47)
      const bool quick_stores = out_bf16 && ldO % 4 == 0 && reinterpret_cast<uintptr_t>(O) % 8 == 0;
      if (fits(2)) {
        if (lists && (wgs(4) >= 384 || wgs(2) > round)) pick = 4;
        else if ((long_stages || !out_bf16) && wgs(2) >= tall && wgs(2) <= round) pick = 2;
      } else if (fits(1)) {
        if (lists && ((long_stages && wgs(1) > round && !quick_stores) || wgs(3) >= (long_stages ? 448 : 384))) pick = 3;
        else if (long_stages && wgs(1) >= 384 && wgs(1) <= round) pick = 1;
      } else if (fits(0)) {
        if (long_stages && !out_bf16 && m->reg_clusters.max_stages < 16 && wgs(0) >= 512) pick = 0;
      }
    }
    if (pick >= 0 && tsh != 1) {
      share_rv = shapes[pick].rv;
      share_pr = shapes[pick].pr;
    }
    if (share_rv) {
      CW = 128;
      G = 1;
      lgS = 0;
      NC = 8;
      ntiles = (N + 512 / share_rv - 1) / (512 / share_rv);
    }
  }
  // fused convolution on a tap-grouped layout whose image rows tile the 64 columns of a wave:
  // the variant that loads one of the three horizontal taps and builds the others.  Measured on
  // the VGG19 layers: 5-15 % faster for images 8 to 32 pixels wide, slower for 4-pixel-wide ones
  // (every lane is a whole image row there: nothing to share, only the extra instructions).
  const bool taps = conv && !bf16 && rbgp_reg_tap_grouped(m) && e->taps_fn && conv->width >= 8 && 64 % conv->width == 0;
  // fp32, two tile rows per MFMA group: lo/hi pairing of the tile rows (rbgp_mfma_reg_dual.hip) where its
  // busiest SIMD walks fewer stages than the longest cluster of the fixed pairs, and stage lists are not split or there are
  // enough of them, of long stages, for a wave on half of the SIMDs (us, fixed pairs split in two -> this: conv5, 96 images, 768
  // lists, fused 15.4 -> 13.4, 69 images 15.7 -> 13.7; VGG19 layer 9 at 1/4, 72 images, 27.0 -> 22.8).
  bool dual = false, dual_half = false;
  {
    const int tp = tune[RBGP_TUNE_ROW_PAIRING];
    if (tp < 0 || tp > 2) return RBGP_EUNSUPPORTED;
    const bool can = !bf16 && !taps && m->reg_dual.ok && rbgp_reg_dual_kernel(pl.KC) && !tune[RBGP_TUNE_K_SPLIT];
    // (merged rows: the caller's mask repeats its rows too few times for pairs, and its knobs count as on that mask)
    const bool merged = !m->merged.empty();
    if (tp == 2 && (!can || merged)) return RBGP_EUNSUPPORTED;
    dual = can && (tp == 2 || (tp == 0 && (lgS == 0 || (by_walk && lists > 512)) && m->reg_dual.max_stages < m->reg_clusters.max_stages &&
                               !(merged && tune[RBGP_TUNE_REGISTER_SETS])));
    dual_half = dual && tp == 0 && lists < 1024;   // (in place of fixed pairs split in two)
  }
  if (dual) lgS = 1;   // (two column tiles per workgroup, as with a stage list split in two)
  // The first call makes the tables of every kernel that a batch of another size takes (it may come under capture; the fused
  // convolution's batch is part of its geometry): fp32 those of the clusters also where tile rows are paired, bf16 those of all groups.
  RegTables *tab = bf16 ? &st->tab_bf16[G == 4 ? 2 : G == 2 ? 1 : 0] : &st->tab;
  auto make_tables = [&](int groups, RegTables *t) { return t->stages ? RBGP_OK : build_tables(m, groups * pl.MG, t); };
  int rc_tables = dual && conv ? RBGP_OK : make_tables(G, tab);
  if (!rc_tables && two_groups) rc_tables = make_tables(1, &st->tab_bf16[0]);
  if (!rc_tables && two_groups) rc_tables = make_tables(2, &st->tab_bf16[1]);
  if (!rc_tables && four_groups && !st->g4_none) {
    rc_tables = make_tables(4, &st->tab_bf16[2]);
    if (rc_tables == RBGP_EUNSUPPORTED && G != 4) {   // (too long a list, which this batch does not walk)
      st->g4_none = true;
      rc_tables = RBGP_OK;
    }
  }
  if (rc_tables) return rc_tables;
  if (dual || share_rv) halves = false;
  if (!dual) {
    // a stage list longer than a wave's table is split over enough waves of the workgroup
    int need = 0;
    while ((kRegWaveStages << need) < tab->max_stages) ++need;
    if (need > lgS) {
      if (tune[RBGP_TUNE_K_SPLIT]) return RBGP_EUNSUPPORTED;
      lgS = need;
      halves = false;
    }
  }
  // fp32, rows of G_r moved into the tile-row index: NG of the `fold` tile rows that share their tiles per wave
  // (see spmm_reg), as many as still leave every SIMD a wave; tuning knob RBGP_TUNE_ROW_GROUPS overrides.
  int NGf = 1;
  const RegGroupEntry *ge = nullptr;
  // fp32 on the bf16 matrix core (rbgp_mfma_reg_split.hip): waves of two tile rows and 128 columns, each by itself
  // (split_rw = 1) or four of them sharing the columns (4)
  int split_rw = 0;
  bool sparse = false;   // those that share columns: the sparse MFMA
  {
    const int tsp = tune[RBGP_TUNE_SPLIT_OPERANDS];
    if (tsp < 0 || tsp > 3) return RBGP_EUNSUPPORTED;
    const bool knobs = tune[RBGP_TUNE_ROW_GROUPS] || tune[RBGP_TUNE_COLUMN_TILES] || tune[RBGP_TUNE_REGISTER_SETS];
    const int64_t tiles = (N + 127) / 128, waves = int64_t(pl.TR / 2) * m->a[2] * tiles;
    const bool can = !bf16 && !dual && ident && !knobs && pl.fold % 2 == 0;
    // (waves that share columns pass a barrier per round: no split stage lists)
    sparse = !conv && !m->pairs.empty();
    const bool can4 = can && pl.fold % 8 == 0 && tab->max_stages <= kRegWaveStages && !tune[RBGP_TUNE_K_SPLIT];
    if ((tsp == 2 && !can) || (tsp == 3 && !can4)) return RBGP_EUNSUPPORTED;
    // waves of a list: enough for two per SIMD, while each keeps four blocks of 16 steps to amortise its start and stores;
    // a split in two that leaves a fifth of those places empty is better than one in four that needs a second round for
    // them (us, in two / in four: L2 at 112 images 25.5 / 28.4, L3 41.2 / 44.8; 1/16, four rows, N = 896 35.8 / 37.8)
    const int64_t blocks = int64_t(tab->max_stages) * ((pl.KCR + 15) / 16);
    int lg = 0;
    while (lg < 2 && ((kRegWaveStages << lg) < tab->max_stages ||
                      ((waves << lg) < (lg == 1 ? 1600 : 2048) && (blocks >> (lg + 1)) >= 4))) ++lg;
    if (tsp >= 2) {
      split_rw = tsp == 2 ? 1 : 4;
    } else if (tsp == 0 && can && rbgp_reg_split_cycles(m) < rbgp_reg_fp32_cycles(m)) {
      // Measured against the fp32 MFMA kernels (us, fp32 -> waves by themselves / sharing): 4096^3 at density 1/4, one
      // row per column set, N = 4096 514 -> 409 / 337, 1531 207 -> 166 / 152, 1000 140 -> 112 / 116, 512 77 -> 64 / 102,
      // 256 44 -> 40 / 101, 64 14.4 -> 35 / 100 (sparse MFMA: 75 up to 1024, by themselves 57 at 512, 82 at 640); 1/16, four
      // rows, N = 4096 174 -> 120 / 90, 256 15.3 -> 14.9 / 30; VGG19 layers at density 1/2 forward 30.2 -> 25.1 (L2), 52.9 -> 44.6 (L3), 16.1 -> 40.3 (L13: 256 waves).  So: sharing from
      // five workgroups per four CUs on, with the sparse MFMA from five per eight; by themselves where every SIMD gets two
      // waves, or one with a long list.  Where it takes a split in four to reach exactly that many waves, the fp32 kernels, whose waves are half as wide, run one full
      // round: stages of 72 or 64 steps then stay there (us, fp32 -> waves by themselves: L6 at 64 images 24.2 -> 27.0, at
      // 80 40.5 -> 37.5; L9 at 128 46.0 -> 47.1; one tile column, 64 steps, N = 256 23.9 -> 24.7), as do the shortest lists
      // (L2 at 64 images, 20 blocks, 16.5 -> 17.0, at 80 27.5 -> 23.8), but not stages of 32 steps (1/4, one row, N = 256
      // 43.2 -> 40.4) nor lists of 32 blocks and more (L3 at 64 images 27.9 -> 26.4; 1/16, four rows, N = 512 24.4 -> 22.7).
      const int64_t enough = blocks >= 64 ? 1024 : lg == 1 ? 1600 : 2048;
      const bool full_round = (waves << 2) == enough && (blocks >= 64 ? pl.KC > 36 : blocks < 32);
      // Short lists of 32-step stages (transposed layers at 1/2), whose fp32 waves cost mostly latency, two of them on a SIMD
      // little more than one: 8 blocks only where lists stay whole (L6 at 32 images, split in two, 19.6 -> 21.9), and not with
      // a second round half empty (L6 at 64 images 30.7 -> 29.9, at 80 40.0 -> 45.5, 96 42 -> 45.8, 112 50.3 -> 47.2, 128
      // 54 -> 47.5); 16 blocks not where only these kernels need a second round (L8 at 64 images 21.1 -> 20.3, 72 to 112
      // 21-22.7 -> 28.4-30, 128 31.5 -> 30.8).
      bool late_round = false;
      if (pl.KC <= 32 && blocks > 4 && blocks < 32) {
        const int64_t fp32_waves = int64_t(pl.TR / 2) * m->a[2] * ((N + 63) / 64);
        late_round = blocks < 16 ? lg > 0 || (waves > 2304 && waves < 3840)
                                 : fp32_waves <= 1024 ? (waves << lg) > 2048 : fp32_waves <= 2048 && (waves << lg) > 2304;
      }
      if (can4 && waves / 4 >= (sparse ? 160 : 320))
        split_rw = 4;
      else if ((waves << lg) >= enough && !full_round && !late_round)
        split_rw = 1;
    }
    if (split_rw) {
      ntiles = tiles;
      if (split_rw > 1) lgS = 0;
      else if (!tune[RBGP_TUNE_K_SPLIT]) lgS = lg;
    }
  }
  const bool split = split_rw > 0;
  if (!bf16 && sparse && !st->pairs) {   // (with the first call, whatever N: a wider batch may come under capture)
    int rc = upload(m->pairs, &st->pairs);
    if (rc) return rc;
  }
  if (!bf16 && !dual && !split && pl.MG == 1 && pl.fold > 1) {
    auto fits = [&](int ng) {
      const RegGroupEntry *g = find_reg_groups(pl.KC, ng);
      return ident && pl.fold % ng == 0 && g && (!taps || g->taps_fn);
    };
    const int tg = tune[RBGP_TUNE_ROW_GROUPS];
    if (tg > 1) {
      if (!fits(tg)) return RBGP_EUNSUPPORTED;
      NGf = tg;
    } else if (tg == 0) {
      // (not for short waves: with several groups a SIMD holds one wave instead of up to four, and a wave of a few
      // hundred MFMAs is mostly latency -- the conv5 backward data product, 8 stages of 8 steps: 29.6 us with one
      // group, 39.8 / 35.3 with two / four; the density-1/2 VGG19 layers, 8-16 stages of 72 steps: 6-19 % faster with two)
      const int64_t steps = int64_t(tab->max_stages) * pl.KC;
      for (int ng : {4, 2})
        if (fits(ng) && steps >= (128 * ng << lgS) && ((int64_t(tab->ncl / ng) * m->a[2] * ntiles) << lgS) >= 1024) {
          NGf = ng;
          break;
        }
      // (the kernels of two groups with stages of up to 32 steps fit two waves per SIMD, like those of one group or
      // nearly so: there two groups pay from 64 steps on, while every SIMD still gets its two waves)
      if (NGf == 1 && fits(2) && pl.KC <= 32 && !taps && steps >= (64 << lgS) &&
          ((int64_t(tab->ncl / 2) * m->a[2] * ntiles) << lgS) >= 2048)
        NGf = 2;
    }
    if (NGf > 1) ge = find_reg_groups(taps || NGf > 2 ? pl.KC : walk, NGf);
  } else if (!bf16 && !split && tune[RBGP_TUNE_ROW_GROUPS] > 1) {
    return RBGP_EUNSUPPORTED;
  }
  // fp32, stages of up to 8 steps (short waves, mostly latency): column tiles per wave (see spmm_reg); tuning knob
  // RBGP_TUNE_COLUMN_TILES overrides.
  int CT = 1;
  {
    const int tc = tune[RBGP_TUNE_COLUMN_TILES];
    bool can = !bf16 && !dual && !split && !conv && find_reg_tiles(pl.KC, pl.RS, NGf) && lgS == 0 && tab->max_stages > 0 && tab->max_stages % 4 == 0 &&
               m->reg_clusters.U == pl.MG;
    for (size_t c = 0; can && c < m->reg_clusters.counts.size(); ++c) can = m->reg_clusters.counts[c] == tab->max_stages;
    auto fits = [&](int c) { return can && (c == 2 || c == 4 || c == 8) && tab->max_stages * c <= kRegWaveStages; };
    auto waves = [&](int ng, int c) { return int64_t(tab->ncl / ng) * m->a[2] * ((ntiles + c - 1) / c); };
    if (tc > 1) {
      if (!fits(tc)) return RBGP_EUNSUPPORTED;
      CT = tc;
    } else if (tc == 0 && NGf == 2) {
      for (int c : {4, 2})
        if (fits(c) && waves(2, c) >= 2048) {
          CT = c;
          break;
        }
    } else if (tc == 0 && NGf == 1) {
      // Measured on the conv5 backward data product (64 tile rows of 9 rows, 8 stages of 8 steps, 16 384 such
      // waves), us per launch on one box: one tile per wave 31.2, four 29.6; two of the tile rows that share their
      // tiles per wave as well (each row of dO loaded half as often; two waves per SIMD) 27.8 with four tiles, 28.8
      // with two, 32.4 with eight.  The waves must still fill the SIMDs: three each with one row group, two with two.
      if (tune[RBGP_TUNE_ROW_GROUPS] == 0 && ident && pl.fold % 2 == 0 && find_reg_tiles(pl.KC, pl.RS, 2) && fits(4) &&
          waves(2, 4) >= 2048) {
        NGf = 2;
        CT = 4;
      } else {
        for (int c : {4, 2})
          if (fits(c) && waves(1, c) >= 3072) {
            CT = c;
            break;
          }
      }
    }
  }
  // One register set with more waves per SIMD instead of two sets (see spmm_reg, spmm_reg_bf16) wherever that variant
  // is built; tuning knob RBGP_TUNE_REGISTER_SETS overrides.
  bool lean = false;
  {
    const int tr = tune[RBGP_TUNE_REGISTER_SETS];
    if (tr < 0 || tr > 2) return RBGP_EUNSUPPORTED;
    // (bf16, two groups of short stages: only where a wave has a single stage -- nothing to prefetch, so the second set
    // buys nothing and the extra waves do, 27.6 -> 22.2 us on the dense first VGG19 layer; with several short stages
    // the two sets keep more bytes in flight, 18.5 against 23.6 us on layer 2 at density 1/8)
    const bool can = share_rv ? false
                     : bf16   ? rbgp_reg_bf16_lean_kernel(pl.KC, pl.RS, G, CW) != nullptr &&
                                (pl.KC > 32 || G == 4 || tab->max_stages <= (1 << lgS))
                          : !dual && !split && CT == 1 && find_reg_lean(taps ? pl.KC : walk, pl.RS, taps, NGf);
    if (tr == 1 && !can) return RBGP_EUNSUPPORTED;
    // (measured on the fp32 VGG19 layers at every density, batches of 512 to 131 072 columns, split lists included:
    // stages of 72 steps 1-19 % faster than two sets in every cell, the shorter stages and the tap-grouped kernels
    // 1-2 % over the forward, fused and backward sweeps (single cells up to 12 %); bf16 on 128-column tiles: 1-13 %
    // faster in 38 of 41 cells, 2-6 % slower in three; so it is the default wherever it applies)
    lean = can && tr != 2;
  }
  const int ncl = dual ? m->reg_dual.nq : split ? tab->ncl / (2 * split_rw) : share_rv ? tab->ncl / (2 * share_rv * share_pr) : tab->ncl / NGf;
  const int fpm = m->d[0] * pl.NSTG;
  // LDS: partial sums of the split -- per wave the (S - 1) / S of its 4G units it does not own; lo/hi pairing:
  // the four units of half of the eight waves
  size_t lds = dual ? size_t(16) * 1024
                    : size_t(4) * ((4 * G) >> lgS) * ((1 << lgS) - 1) * (bf16 ? NC / 4 : 1) * 1024;
  if (split_rw == 1) lds = size_t(4) * (16 >> lgS) * ((1 << lgS) - 1) * 1024;
  if (split_rw > 1 || share_rv) lds = 0;   // (static)
  lds *= NGf;   // (fp32 with several groups per wave: one such block per group)

  RegParams rp;
  rp.Wp = static_cast<const float *>(packed);
  rp.I = static_cast<const float *>(I);
  rp.O = static_cast<float *>(O);
  rp.obf16 = out_bf16 ? 1 : 0;
  // Stores past the caches, but not of rows that begin inside a segment of 64 bytes where O fills most of the Infinity Cache: the parts of a
  // segment that two workgroups write meet in memory, and wait for one another there (us, a store an element / past the caches / through
  // them: transposed WRN group 1, 112 MB of O 57.6 / 54.6 / 42.5, 160 MB 80.5 / 81.1 / 59.4, transposed layer 3 at 1/8, 24673 columns 59.8 / 62.9 /
  // 43; 80 MB 43.1 / 38.3, through them 32 to 38; 240 MB, which nothing holds, 145 / 109 / 120).
  const int64_t mb = m->M * N * 4 >> 20;
  rp.through = mb >= 96 && mb < 192 && (ldO % 16 || reinterpret_cast<uintptr_t>(O) % 64);
  rp.rowtab = *rowtab;
  rp.stages = dual ? nullptr : tab->stages; rp.counts = dual ? nullptr : tab->counts; rp.members = dual ? nullptr : tab->members;
  rp.tstride = tab->tstride;
  rp.N = N; rp.ldI = ldI; rp.ldO = ldO;
  rp.w_bytes = uint32_t(w_bytes);
  rp.row_bytes = uint32_t(ldI * es);
  rp.n_bytes = uint32_t((bf16 ? (N + NC - 1) / NC * NC : N) * es);
  rp.last_row = int(m->K - 1);
  rp.src_rows = pl.SRC;
  rp.colbase = nullptr;
  if (conv) {
    // pixel offset of every group of NC columns (one lane's load), padded to whole wave tiles with a
    // pixel inside X; fp32: bit 0 / bit 1 flag a group at the left / right border of its image row
    int32_t **cbt = &st->colbase[bf16][CW == 128];
    if (!*cbt) {
      const int64_t H = conv->height, W = conv->width;
      std::vector<int32_t> cb(size_t((N + 511) / 512) * (512 / NC), int32_t((W + 3) * es));
      for (int64_t n = 0; n < N; n += NC) {
        const int64_t img = n / (H * W), y = (n % (H * W)) / W, x = n % W;
        int32_t v = int32_t(((img * (H + 2) + y + 1) * (W + 2) + x + 1) * es);
        if (!bf16) v |= (x == 0 ? 1 : 0) | (x + 4 == W ? 2 : 0);
        cb[size_t(n / NC)] = v;
      }
      int rc = upload(cb, cbt);
      if (rc) return rc;
    }
    rp.colbase = *cbt;
  }
  rp.conv = conv ? 1 : 0;
  rp.conv_h = conv ? int(conv->height) : 0;
  rp.conv_w = conv ? int(conv->width) : 0;
  if (conv) {   // the unit of the stage descriptors is a channel of X
    rp.row_bytes = uint32_t(chs);
    rp.n_bytes = uint32_t(chs);
    rp.last_row = int(m->K / 9 - 1);
    rp.src_rows = pl.SRC / 9;
  }
  rp.a2 = pl.A2; rp.a3 = m->a[2]; rp.a4 = m->a[3]; rp.R = pl.R;
  rp.fpm = fpm;
  rp.pairs = st->pairs; rp.fold = pl.fold;
  rp.tm = pl.A2 * m->a[2] * m->a[3];
  rp.no4 = bf16 ? 32 * rbgp_bf16_blocks32(pl.KC) + (rbgp_bf16_tail16(pl.KC) ? 16 : 0) : pl.NO * 4;
  rp.kcr = pl.KCR;
  rp.frag_bytes = bf16 ? (rbgp_bf16_blocks32(pl.KC) + (rbgp_bf16_tail16(pl.KC) ? 1 : 0)) * 4 * pl.RS * 16 : pl.NQ * 4 * pl.RS * 16;
  rp.nq = bf16 ? (pl.KCR + 31) / 32 : (pl.KCR + 15) / 16;
  for (int r = 0; r < 16; ++r) rp.rowofs[r] = (r / m->a[3]) * m->a[2] * m->a[3] + r % m->a[3];
  rp.ntiles = int(ntiles);
  rp.lgS = lgS;
  const int64_t tiles_per_wg = split_rw > 1 ? 1 : share_rv ? 1 : (4 >> lgS) * CT;
  rp.ct = CT;
  rp.ct_cnt = tab->max_stages;
  rp.by_ct_cnt = rbgp_fast::div_by(std::max(1, rp.ct_cnt));
  const int64_t nquads = (ntiles + tiles_per_wg - 1) / tiles_per_wg;
  // one-dimensional grid, items dealt to the XCDs in blocks (see RegParams)
  // (measured on one box, us: conv5 18.0 / 18.2 / 18.2 with order 1 / 0 / 2; conv3 bf16 20.2 / 17.8 / 17.6; WRN 90.9 / 76.4 / 75.9)
  rp.order = (m->e[2] == 1 && nquads <= 64) ? 1 : nquads >= 8 ? 2 : 0;
  const int64_t items = int64_t(ncl) * m->a[2] * nquads;
  const int64_t per_xcd = rp.order == 2 ? int64_t(ncl) * m->a[2] * ((nquads + 7) / 8) : (items + 7) / 8;
  if (per_xcd * 8 > 0x7fffffff) return RBGP_EUNSUPPORTED;
  rp.ncl = ncl;
  rp.per_xcd = int(per_xcd);
  rp.ngroups = int(nquads);
  set_grid(&rp);
  // Many rows per tile, one stage of 32 rows of I with two of every four kept (transposes of lowered 3x3 layers): workgroups
  // of all rows of a row of G_o x 64 columns (rbgp_mfma_reg_rows.hip), from five workgroups per eight CUs on (us, the kernels
  // above -> this one: VGG19 layer 6 at 1/4, 128 workgroups 8.9 -> 9.6, 192 13.6 -> 10.0, 256 15.3 -> 10.4, 512 26.9 -> 17.4;
  // layer 9, 128 14.0 -> 14.0, 192 22.2 -> 14.8; layer 3, 128 6.6 -> 8.2, 256 10.2 -> 8.5), where groups of 32 rows are nearly
  // full (layer 2: 72 rows, 31.5 -> 31.2).  Not lists of up to two stages in 17 to 23 column tiles, which leave some XCDs half as
  // many workgroups again as others and CUs two (layer 9 at 1/16: 16 tiles 9.8 -> 8.3, 17 11.6 -> 13.6, 20 11.7 -> 12.7, 22
  // 12.9 -> 12.8 to 13.6, 24 13.0 -> 13.0, 25 15.1 -> 13.7), nor on a CU each in 17 to 20, which spmm_reg walks a sixth faster than 21
  // (layers 5-7 at 1/8: 20 tiles 7.6 -> 8.3, 21 9.0 -> 8.4, 24 9.0 -> 8.5).
  const int rows_wg = pl.fold * m->a[2] * pl.R, groups = (rows_wg + 31) / 32;
  if (!bf16 && !conv && !dual && in_order && pl.VC == 4 && pl.NSTG == 1 && m->c[2] == 4 && m->d[2] == 2 && m->c[3] == 2 && m->d[3] == 2 &&
      tab->max_stages <= 12 && 8 * groups * 32 <= 9 * rows_wg && groups <= 64 && !tune[RBGP_TUNE_ROW_GROUPS] && !tune[RBGP_TUNE_K_SPLIT] &&
      !tune[RBGP_TUNE_COLUMN_TILES] && !tune[RBGP_TUNE_REGISTER_SETS] && !tune[RBGP_TUNE_SPLIT_OPERANDS]) {
    const int64_t rows_o = pl.TR / pl.fold, tiles64 = (N + 63) / 64, tiles96 = (N + 95) / 96, all = tiles64 * rows_o;
    auto launched = [&](int64_t tiles) { return rows_o * (tiles >= 8 ? 8 * ((tiles + 7) / 8) : tiles); };
    // 96 columns where 64 give some CUs a second workgroup and 96 none (us, 64 columns -> 96: layers 5-7 at 1/4, 296 workgroups
    // 16.2 -> 13.6, 384 16.4 -> 13.8; layers 5-7 at 1/8, 296 13.5 -> 11.9; layer 9 at 1/16, 384 13.2 -> 11.6); not beyond: a
    // workgroup of 96 takes a quarter to a third longer than one of 64 (layer 6 at 1/4: 192 workgroups of 64 10.2, 128 of 96 13.0;
    // 512 of 64 16.7, 344 of 96 23.9).
    const bool uneven = tab->max_stages <= 2 && (all > 256 ? tiles64 < 24 : tiles64 > 16 && tiles64 <= 20);
    const bool wide = !uneven && tab->max_stages <= 4 && all > 256 && launched(tiles96) <= 256;
    const int64_t tiles = wide ? tiles96 : tiles64, wgs = launched(tiles);
    const size_t bytes = size_t(tab->max_stages) * (wide ? 18432 : 12288) + size_t(groups) * 512;
    const bool far = (int64_t(rows_wg) * ldO + 128) * 4 >= (int64_t(1) << 32);   // (else 32-bit offsets into a workgroup's rows of O)
    if (all >= 160 && !uneven && wgs <= 0x7fffffff && bytes <= 160 * 1024) {
      rp.ntiles = int(tiles);
      rp.ncl = int(rows_o);
      rp.order = tiles >= 8 ? 2 : 0;
      set_grid(&rp);
      rp.by_row = rbgp_fast::div_by(int64_t(rp.a3) * rp.R); rp.by_r = rbgp_fast::div_by(rp.R); rp.by_a4 = rbgp_fast::div_by(rp.a4);
      rp.ct_cnt = tab->max_stages;
      // A wave per group while every workgroup has a CU to itself, or lists are longer than four stages (eight: LDS holds one
      // workgroup, 4 waves 36, 9 waves 27 at 512 workgroups; five and six: two of four waves fit, nine leave registers for
      // one, 4 waves / 9: six stages, 592 workgroups 33.9 / 31.9, 1024 40.9 / 44.9, five, 296 18.3 / 19.7, 768 32.3 / 30.8);
      // else four waves, three workgroups a CU (layer 6: 4 waves / 9, 256 workgroups 14.1 / 10.4, 296 16.5 / 18.1, 768 21.4 /
      // 27.0).
      const int waves = wide || all <= 256 || tab->max_stages > 4 ? std::min(groups, 9) : 4;
      reg_fn rows = rbgp_reg_rows_kernel(wide ? 3 : 2, far);
      if (bytes > 64 * 1024)
        RBGP_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(rows), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)));
      hipLaunchKernelGGL(rows, dim3(unsigned(wgs)), dim3(unsigned(64 * waves)), bytes, static_cast<hipStream_t>(stream), rp);
      RBGP_HIP(hipGetLastError());
      if (far) rbgp_set_last_kernel("spmm_reg_rows", {wide ? 3 : 2, 1});
      else rbgp_set_last_kernel("spmm_reg_rows", {wide ? 3 : 2});
      return RBGP_OK;
    }
  }
  // Few columns: workgroups of 16 columns whose eight waves share a list (rbgp_mfma_reg_narrow.hip), while each has a CU, or with stages
  // of up to 36 steps half of one.  us, spmm_reg / this one, VGG19: layer 13 at 1/2 (32 lists of 72-step stages), 16 columns 12.3 / 5.8, 128
  // (256 workgroups) 13.0 / 10.7, 256 13.6 / 16.7; at 1/4 10.2 / 5.2, 10.5 / 7.9, 11.0 / 11.1; at 1/16 6.1 / 3.9, 6.1 / 4.2, 6.4 / 6.6; layer
  // 6 at 1/4 (16 lists), 64 columns 6.0 / 4.1, 256 6.1 / 4.3, 512 6.4 / 7.1; layer 9 fused at 1/4, 128 9.5 / 7.2, 256 10.0 / 9.3; transposes,
  // stages of 18 and 32 steps: layer 13 at 1/4 (384 lists), 16 columns 5.3 / 3.9, 32 5.3 / 5.0, 64 5.3 / 7.8; layer 8 at 1/2 (144), 32
  // 4.7 / 4.0, 64 4.7 / 5.1.  bf16 (spmm_reg_bf16 with one row group on 64 columns): layer 13 at 1/2, 4 columns 9.9 / 4.6, 128 10.2 / 8.0; at 1/4
  // 64 8.0 / 5.5, 128 8.2 / 6.3; layer 8 fused at 1/2, 64 8.0 / 4.0; gradients of layer 8 at 1/2, 32 columns 10.0 / 9.2 (both).
  if ((bf16 ? G == 1 && CW == 64 && !share_rv && !tune[RBGP_TUNE_COLS_PER_WORKGROUP] : !dual && !split && NGf == 1 && CT == 1) && !tune[RBGP_TUNE_K_SPLIT] && !tune[RBGP_TUNE_ROW_GROUPS] &&
      !tune[RBGP_TUNE_REGISTER_SETS] && !tune[RBGP_TUNE_COLUMN_TILES]) {
    const int64_t tiles = (N + 15) / 16, lists = int64_t(ncl) * m->a[2];
    reg_fn narrow = lists * tiles <= (pl.KC > 36 ? 256 : 512) ? rbgp_reg_narrow_kernel(pl.KC, pl.RS, bf16) : nullptr;
    if (narrow) {
      rp.ntiles = rp.ngroups = int(tiles);
      rp.order = (m->e[2] == 1 && tiles <= 64) ? 1 : tiles >= 8 ? 2 : 0;
      rp.per_xcd = int(rp.order == 2 ? lists * ((tiles + 7) / 8) : (lists * tiles + 7) / 8);
      set_grid(&rp);
      hipLaunchKernelGGL(narrow, dim3(unsigned(8 * rp.per_xcd)), dim3(512), 0, static_cast<hipStream_t>(stream), rp);
      RBGP_HIP(hipGetLastError());
      rbgp_set_last_kernel("spmm_reg_narrow");
      return RBGP_OK;
    }
  }
  reg_fn fn = dual     ? nullptr
              : share_rv ? rbgp_reg_bf16_shared_kernel(share_rv, share_pr)
              : bf16   ? (halves ? rbgp_reg_bf16_half_kernel(walk, pl.RS, CW) : lean ? rbgp_reg_bf16_lean_kernel(G < 4 ? walk : pl.KC, pl.RS, G, CW) : rbgp_reg_bf16_kernel(G < 4 ? walk : pl.KC, pl.RS, G, CW))
              : split  ? rbgp_reg_split_kernel(split_rw, sparse)
              : CT > 1 ? find_reg_tiles(pl.KC, pl.RS, NGf)
              : halves && NGf == 1 ? find_reg_half(taps ? pl.KC : walk, pl.RS, taps)
              : lean   ? find_reg_lean(taps ? pl.KC : walk, pl.RS, taps, NGf)
              : ge   ? (taps ? ge->taps_fn : ge->global_fn)
              : taps ? e->taps_fn
                     : e->global_fn;
  if (!fn && !dual) return RBGP_EUNSUPPORTED;
  if (lds > 64 * 1024 && fn)   // (cheap host-side call; repeated because fn varies with the knobs)
    RBGP_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 int(lds)));
  if (dual) {
    DualParams dq;
    dq.r = rp;
    const DualLayout l = dual_layout(m);
    dq.rt_stride = l.np4; dq.cmax = l.cmax; dq.o_stages = l.stages; dq.o_quads = l.quads;
    dq.tab = *rowtab + l.first;
    rbgp_dual_fn dfn = dual_half ? rbgp_reg_dual_half_kernel(pl.KC) : rbgp_reg_dual_kernel(pl.KC);
    hipLaunchKernelGGL(dfn, dim3(unsigned(8 * per_xcd)), dim3(512), lds, static_cast<hipStream_t>(stream), dq);
  } else {
    hipLaunchKernelGGL(fn, dim3(unsigned(8 * per_xcd)), dim3(256), lds, static_cast<hipStream_t>(stream), rp);
  }
  RBGP_HIP(hipGetLastError());
  if (dual) rbgp_set_last_kernel("spmm_reg_dual");
  else if (share_rv) rbgp_set_last_kernel("spmm_reg_bf16_shared", {share_rv, share_pr});
  else if (split_rw > 1) rbgp_set_last_kernel("spmm_reg_split_shared", {sparse});
  else if (split) rbgp_set_last_kernel("spmm_reg_split");
  else rbgp_set_last_kernel(bf16 ? "spmm_reg_bf16" : "spmm_reg");
  return RBGP_OK;
}
