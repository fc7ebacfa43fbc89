// The weight gradient's MFMA kernel for most shapes (see rbgp_sddmm.hip for its units): eight waves per workgroup, two per
// SIMD, each with its own range of the batch, RB groups of 16 rows of dO and NB groups of 16 rows of I; a step is 128 bytes
// of a row, one cache line: 32 columns in fp32, 64 in bf16.  Compared with sddmm_reg (steps of 64 bytes, four waves, whole
// stages): twice the bytes in flight, lines asked for once, a unit's outputs split over workgroups before the batch is (no
// partial sums, no second launch), the workgroups of an XCD chosen for the rows they share.
// CONV: the three horizontal taps of a channel row are one window of a lane's columns and one pixel to either side (16 bytes and 4
// or 8 more, aligned to 4 bytes): a third of the rows of sddmm_reg, whose bf16 loads are mostly aligned to 2 bytes.  Stages of
// 36 steps and more (WIN) pass the window through LDS once and make the taps from it in registers, so that fp32 splits it once:
// 194 vector instructions a step for 2 x 3 groups, where three shifted copies of the rows took 260 (and 1.4 times the LDS traffic,
// in bf16 1.8 times).  Shorter stages, whose windows do not fill a group, write it three times, shifted.
// fp32: operands are split (rbgp_split.h) after the pass through LDS, and their products go through the bf16 matrix core: 6.5
// vector instructions a value, 36 MFMAs of 16 cycles instead of 48 of 32 for 2 x 3 groups x 32 columns.
//
// us, before (sddmm_reg, with its second launch) -> this kernel, lowered: VGG19 conv3 bf16, 8192 columns 20.5 -> 15.5, 2368 13.0
// -> 8.2; layer 6 at 1/4 fp32, 2368 columns 19.1 -> 16.3, 320 columns 10.9 -> 6.7; fused, shifted copies / windows: conv3 bf16
// 19.0 -> 13.7 / 11.6, WRN group 1 bf16 27.9 -> 21.2 / 18.5, conv5 fp32 23.2 -> 19.0 / 16.5, layer 6 at 1/4 fp32, 2368 columns
// 18 -> 16.3 / 12.8; fp32 error against 64-bit sums 1.8e-7 -> 0.8e-7.
// What bounds it (conv5 fp32 fused, timing-only builds of the shifted copies): empty loops 5.3 (launch, tables, adding up eight waves),
// the loads alone 11 (lowered 13.4: memory), the passes through LDS alone 12.5, loads and LDS 14.5.  Tried: twelve waves (23.2,
// spills), four (25), one step in flight (21.1), fp32 MFMAs (22.5), each workgroup's steps starting elsewhere in its range (no
// change); lowered, buffer loads with scalar column offsets, 30 of 280 vector instructions a step fewer (no change).
#include <hip/hip_runtime.h>

#include "rbgp_sddmm.h"
#include "rbgp_split.h"

using namespace rbgp_split;
using rbgp_sddmm_detail::SddmmParams;

namespace {

constexpr int kWaves = rbgp_sddmm_detail::kLinesWaves;
typedef u32x4 u32x4_u __attribute__((aligned(4)));
typedef bf16x8 bf16x8_any __attribute__((aligned(2)));

template <bool BF16>
struct Operand;
// fp32: the parts of the split operands (rbgp_split.h) go through v_mfma_f32_16x16x32_bf16, the product of the leading
// parts into one accumulator and the five small ones into another; `again` is the fp32 form, for sums that are not finite.
template <>
struct Operand<false> {
  static constexpr int CPL = 4;   // columns per lane and load
  static constexpr int WX = 2;    // dwords of a window past a lane's 16 bytes
  static __device__ __forceinline__ u32x4 load_any(const unsigned char *at) {
    return *reinterpret_cast<const u32x4_u *>(at);
  }
  // moved down by s columns (1 to 3), zeros behind
  static __device__ __forceinline__ u32x4 moved(u32x4 x, int s) {
    x = s & 1 ? u32x4{x[1], x[2], x[3], 0} : x;
    return s & 2 ? u32x4{x[2], x[3], 0, 0} : x;
  }
  typedef Split frag;             // operand of 16 rows x 32 columns
  static __device__ __forceinline__ frag make(const u32x4 &lo, const u32x4 &hi) {
    const float x[8] = {__uint_as_float(lo[0]), __uint_as_float(lo[1]), __uint_as_float(lo[2]), __uint_as_float(lo[3]),
                        __uint_as_float(hi[0]), __uint_as_float(hi[1]), __uint_as_float(hi[2]), __uint_as_float(hi[3])};
    return split8(x);
  }
  // the operands of the three horizontal taps, from the lane's two windows of six columns (split once)
  static __device__ __forceinline__ void windows(frag (&f)[3], const u32x4 (&b)[2], const uint32_t (&w)[2][WX]) {
    u32x4 o[3][3];                // [tap][part]
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t p[3][3];           // [pair of columns][part]
      split2(__uint_as_float(b[h][0]), __uint_as_float(b[h][1]), p[0]);
      split2(__uint_as_float(b[h][2]), __uint_as_float(b[h][3]), p[1]);
      split2(__uint_as_float(w[h][0]), __uint_as_float(w[h][1]), p[2]);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        o[0][k][2 * h] = p[0][k];
        o[0][k][2 * h + 1] = o[2][k][2 * h] = p[1][k];
        o[2][k][2 * h + 1] = p[2][k];
        o[1][k][2 * h] = __builtin_amdgcn_alignbit(p[1][k], p[0][k], 16);
        o[1][k][2 * h + 1] = __builtin_amdgcn_alignbit(p[2][k], p[1][k], 16);
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 3; ++k) f[d].p[k] = __builtin_bit_cast(bf16x8, o[d][k]);
  }
  template <int RB>
  static __device__ __forceinline__ void mac(const frag (&a)[RB], const frag &b, f32x4 (&acc)[RB], f32x4 (&cor)[RB]) {
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x4 &d = k == 0 ? acc[rb] : cor[rb];
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb].p[pa[k]], b.p[pb[k]], d, 0, 0, 0);
      }
  }
  static __device__ __forceinline__ void mac_fp32(const u32x4 &a, const u32x4 &b, f32x4 &acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[t]), __uint_as_float(b[t]), acc, 0, 0, 0);
  }
};
template <>
struct Operand<true> {
  static constexpr int CPL = 8;
  static constexpr int WX = 1;
  static __device__ __forceinline__ u32x4 load_any(const unsigned char *at) {   // (any alignment)
    return __builtin_bit_cast(u32x4, *reinterpret_cast<const bf16x8_any *>(at));
  }
  static __device__ __forceinline__ u32x4 moved(u32x4 x, int s) {   // (1 to 7)
    x = s & 1 ? u32x4{__builtin_amdgcn_alignbit(x[1], x[0], 16), __builtin_amdgcn_alignbit(x[2], x[1], 16),
                      __builtin_amdgcn_alignbit(x[3], x[2], 16), x[3] >> 16} : x;
    x = s & 2 ? u32x4{x[1], x[2], x[3], 0} : x;
    return s & 4 ? u32x4{x[2], x[3], 0, 0} : x;
  }
  struct frag {                   // operand of 16 rows x 64 columns
    u32x4 lo, hi;
  };
  static __device__ __forceinline__ frag make(const u32x4 &lo, const u32x4 &hi) { return frag{lo, hi}; }
  // one column up: b[0] and the next of every pair, behind b[3] the first of w
  static __device__ __forceinline__ u32x4 up(const u32x4 &b, uint32_t w) {
    return u32x4{__builtin_amdgcn_alignbit(b[1], b[0], 16), __builtin_amdgcn_alignbit(b[2], b[1], 16),
                 __builtin_amdgcn_alignbit(b[3], b[2], 16), __builtin_amdgcn_alignbit(w, b[3], 16)};
  }
  static __device__ __forceinline__ void windows(frag (&f)[3], const u32x4 (&b)[2], const uint32_t (&w)[2][WX]) {
    f[0] = frag{b[0], b[1]};
    f[1] = frag{up(b[0], w[0][0]), up(b[1], w[1][0])};
    f[2] = frag{u32x4{b[0][1], b[0][2], b[0][3], w[0][0]}, u32x4{b[1][1], b[1][2], b[1][3], w[1][0]}};
  }
  template <int RB>
  static __device__ __forceinline__ void mac(const frag (&a)[RB], const frag &b, f32x4 (&acc)[RB], f32x4 (&)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[rb].lo), __builtin_bit_cast(bf16x8, b.lo),
                                                        acc[rb], 0, 0, 0);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[rb].hi), __builtin_bit_cast(bf16x8, b.hi),
                                                        acc[rb], 0, 0, 0);
  }
};

// RB: groups of 16 rows of dO per wave; NB: groups of 16 contraction steps per wave.  WIN (CONV, NB = 3 and 6): a group is one
// horizontal tap of 16 pixel rows (channel, dy), and the three taps of the same 16 rows (24 with NB = 6) come out of one window.
template <int RB, int NB, bool BF16, bool CONV, bool GI, bool FAR>
__global__ __launch_bounds__(64 * kWaves) void sddmm_lines(SddmmParams p) {
  typedef Operand<BF16> Op;
  constexpr int CPL = Op::CPL, CPI = 8 * CPL;   // columns per lane load / per step: 128 bytes of a row
  constexpr int ES = BF16 ? 2 : 4;
  constexpr bool WIN = CONV && NB >= 3;
  static_assert(!WIN || NB % 3 == 0, "whole windows");
  constexpr int NGB = WIN ? NB / 3 : NB;        // groups of 16 rows of B in LDS
  constexpr int NG = RB + NGB;
  // CONV: pixel rows, three taps each, whose windows one step loads: eight per load instruction
  constexpr int NPL = WIN ? (NB == 6 ? 3 : 2) : (16 * NB + 23) / 24;   // (a stage has at most 72 steps)
  constexpr int NLI = CONV ? NPL : 2 * NB;      // 16-byte loads of rows of I per step
  constexpr int kExtra = WIN ? NGB * 32 * Op::WX : CONV ? 64 : 0;   // ends of windows; without WIN what is past the last step
  constexpr int kTile = NG * 128 + kExtra;      // 16-byte slots of a wave: 16 rows x 128 bytes per group
  __shared__ union {
    u32x4 stage[kWaves][kTile];
    float red[kWaves][RB * NB * 4][64];
  } lds;
  const int lane = threadIdx.x & 63, j = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // load layout: lane l reads rows l / 8 and 8 + l / 8 of the 16, 16-byte segment l % 8; operand layout: lane l holds
  // row l % 16, segments l / 16 and 4 + l / 16 (any order of the columns does, as long as both operands have it)
  const int lr = lane >> 3, ls = lane & 7;
  // a tile in LDS: slot 8 * row + (segment ^ (row & 7)): eight consecutive lanes meet all banks, writing and reading
  const int wslot = 8 * lr + (ls ^ lr);
  const int rslot0 = 8 * j + (q ^ (j & 7)), rslot1 = 8 * j + ((q + 4) ^ (j & 7));
  // (what the prologue reads of the kernel arguments, at once: see grid_args)
  asm volatile("" ::"s"(p.by_halves.mul), "s"(p.by_halves.shift), "s"(p.by_RBG.mul), "s"(p.by_RBG.shift), "s"(p.by_a3.mul),
               "s"(p.by_a3.shift), "s"(p.by_NSTG.mul), "s"(p.by_NSTG.shift), "s"(p.by_c1.mul), "s"(p.by_c1.shift), "s"(p.by_a4.mul),
               "s"(p.by_a4.shift), "s"(p.order), "s"(p.colrows), "s"(p.rowtab), "s"(p.EO), "s"(p.dO), "s"(p.I), "s"(p.ld_dO), "s"(p.R),
               "s"(p.tile_rows), "s"(p.stage_rows), "s"(p.lgRS), "s"(p.MG), "s"(p.chunk), "s"(p.N));
  // Workgroups go to the eight XCDs round-robin in launch order, and each XCD has its own L2: the unit numbers are dealt
  // to the XCDs in eight contiguous runs, so that those of one XCD read few rows (see `order`).
  int x;
  {
    const int total = gridDim.x, xcd = blockIdx.x & 7, each = total >> 3, more = total & 7;
    x = xcd * each + (xcd < more ? xcd : more) + int(blockIdx.x >> 3);
  }
  auto split_off = [&](int n, rbgp_fast::Div by) {   // x = x / n; x % n
    const int q = rbgp_fast::quotient(x, by), r = x - q * n;
    x = q;
    return r;
  };
  const int b0 = split_off(p.halves, p.by_halves) * NB;   // first 16-step group of this workgroup
  const int g = split_off(p.RBG, p.by_RBG);
  int u3 = 0, sg, v1;
  if (p.order == 1) {
    sg = split_off(p.NSTG, p.by_NSTG);
    v1 = split_off(p.c1, p.by_c1);
    if constexpr (!GI) u3 = split_off(p.a3, p.by_a3);
  } else {
    if constexpr (!GI) u3 = split_off(p.a3, p.by_a3);
    sg = split_off(p.NSTG, p.by_NSTG);
    v1 = split_off(p.c1, p.by_c1);
  }
  const int part = x;
  const int RS = 1 << p.lgRS;
  const int32_t *crow = p.colrows + v1 * p.EO, *cpos = p.colpos + v1 * p.EO;
  const int base = v1 * p.tile_rows + sg * p.stage_rows;

  // The wave's columns, and where the first of them start inside a channel: requested with the tables, not behind them.
  const int64_t n_lo = (int64_t(part) * kWaves + wave) * p.chunk;
  const int64_t n_hi = n_lo + p.chunk < p.N ? n_lo + p.chunk : p.N;   // (n_lo may lie past N: empty range)
  const int64_t steps = n_hi > n_lo ? (n_hi - n_lo) / CPI : 0;        // whole steps
  // (past the last step the loads repeat it: in bounds)
  const int64_t n_last = n_lo + (steps - 1) * CPI;
  auto column = [&](int64_t k) {
    const int64_t c = n_lo + k * CPI;
    return c < n_last ? c : n_last;
  };
  // CONV: where this lane's group of columns starts inside a channel (columns are pixels in image order)
  // (in elements: scaled here, a lookup would be waited for where it is made)
  auto pixel = [&](int64_t n) { return CONV ? p.colbase[n / CPL + ls] : 0; };
  int at_first[2] = {0, 0}, at_next[2] = {0, 0};   // pixel of steps 0 and 1; of the step that refills set d next, a round ahead
  if (CONV && steps > 0) {
#pragma unroll
    for (int d = 0; d < 2; ++d) at_first[d] = pixel(column(d));
#pragma unroll
    for (int d = 0; d < 2; ++d) at_next[d] = pixel(column(2 + d));
  }

  // row r16 of row group rb of this workgroup: (row of dO, or -1; its entry of the tile-row list; its u_i)
  struct RowOf { int64_t row; int entry, ui; };
  auto row_of = [&](int rb, int r16) {
    RowOf o{-1, 0, u3};
    int ri;
    if constexpr (GI) {
      const int rho = (g * RB + rb) * 16 + r16, block = rbgp_fast::quotient(rho, p.by_R);
      ri = rho - block * p.R;
      o.entry = rbgp_fast::quotient(block, p.by_a3);
      o.ui = block - o.entry * p.a3;
    } else {
      o.entry = (g * RB + rb) * p.MG + (r16 >> p.lgRS);
      ri = r16 & (RS - 1);
    }
    if (o.entry < p.EO && ri < p.R) {
      const int ra = rbgp_fast::quotient(ri, p.by_a4);
      o.row = ((int64_t(crow[o.entry]) * p.a2 + ra) * p.a3 + o.ui) * p.a4 + (ri - ra * p.a4);
    }
    return o;
  };
  // Byte offsets of this lane's 16 bytes in step 0.  CONV: below 2 GiB (inside X) and 4 GiB (inside dO), checked by the host, and the
  // column of a step is a scalar offset of buffer loads, which costs no vector instruction (on the lowered input no gain, and spills).
  // FAR (CONV): 64-bit offsets into a dO of 4 GiB and more.
  typedef typename std::conditional<CONV && !FAR, uint32_t, int64_t>::type OffA;
  typedef typename std::conditional<CONV, uint32_t, int64_t>::type Off;
  OffA offA[2 * RB];
#pragma unroll
  for (int i = 0; i < 2 * RB; ++i) {
    const int64_t row = row_of(i / 2, lr + 8 * (i % 2)).row;
    offA[i] = OffA((row < 0 ? 0 : row) * p.ld_dO * ES + ls * 16);
  }
  const unsigned char *const bytesA = static_cast<const unsigned char *>(p.dO);
  const unsigned char *const bytesB = static_cast<const unsigned char *>(p.I);
  Off offB[NLI];
  int wslotB[CONV && !WIN ? NPL : 1][3];
  if constexpr (CONV) {
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int kk = 16 * b0 + 3 * (8 * i + lr);           // first tap of the pair (b0 is a multiple of 3)
      const int sr = GI ? (kk < p.src_rows ? kk : 0) : (kk < p.KCR ? p.rowtab[u3 * p.nbt * 16 + kk] : 0);
      const int k = base + sr;                             // channel k / 9, dy = (k % 9) / 3 - 1, dx = -1
      offB[i] = Off((int64_t(k / 9) * p.chan_elems + ((k % 9) / 3 - 1) * p.conv_w2 - 1) * ES);
      if constexpr (!WIN) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int row = 3 * (8 * i + lr) + d;
          wslotB[i][d] = row < 16 * NB ? (RB + row / 16) * 128 + (row % 16) * 8 + (ls ^ (row & 7)) : NG * 128 + lane;
        }
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NLI; ++i) {   // padding steps read row 0 of the stage
      const int b = b0 + i / 2, r = lr + 8 * (i % 2), sr = 16 * b + r;
      const int k = base + (GI ? (sr < p.src_rows ? sr : 0) : (b < p.nbt ? p.rowtab[(u3 * p.nbt + b) * 16 + r] : 0));
      offB[i] = Off(int64_t(k) * p.ldI * ES + ls * 16);
    }
  }
  // Where the lane's sums go, with the tables as well (FAR: before the last barrier, held through the loop the pointers cost <2, 1> the
  // second workgroup on a CU); looked up at the end, row after row, they cost two latencies each.
  float *dst[RB];                               // first of the row's kept values of the stage; nullptr: no such row
  int dst_ui[RB];
  auto find_rows = [&]() {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const RowOf o = row_of(rb, 4 * q + wave % 4);
      // the stage is fragment cpos * NSTG + sg of the row: KCR consecutive kept values
      dst[rb] = o.row < 0 ? nullptr
                          : p.out + int64_t(part) * p.nnz + o.row * p.rowdeg + int64_t(cpos[o.entry] * p.NSTG + sg) * p.KCR;
      dst_ui[rb] = o.ui;
    }
  };
  if constexpr (!FAR) find_rows();
  __amdgpu_buffer_rsrc_t arsrc, xrsrc;
  if constexpr (CONV) {
    if constexpr (!FAR) arsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.dO), 0, -1, kRsrcFlags);
    xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.I), 0, int(p.x_bytes), kRsrcFlags);
  }

  // What one step has in flight.  CONV: the window of CPL + 2 pixels that the three horizontal taps of a lane's columns share.
  struct Raw {
    u32x4 a[2 * RB], b[NLI];
    uint32_t w[CONV ? NPL : 1][Op::WX];
  };
  // (`at`: pixel(n), looked up by the caller -- ahead of time inside the loop, where a lookup right before its use
  // would have to wait for every load in flight)
  auto load_all = [&](Raw &r, int64_t n, int at) {
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) {
      if constexpr (CONV && !FAR) r.a[i] = __builtin_amdgcn_raw_buffer_load_b128(arsrc, int(offA[i]), int(uint32_t(n) * ES), 0);
      else r.a[i] = *reinterpret_cast<const u32x4_u *>(bytesA + offA[i] + n * ES);
    }
#pragma unroll
    for (int i = 0; i < NLI; ++i) {
      if constexpr (CONV) {
        const int o = int(offB[i]) + at * ES;
        r.b[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, o, 0, 0);
        if constexpr (BF16) {
          r.w[i][0] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, o, 16, 0);
        } else {
          const auto w = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, o, 16, 0);
          r.w[i][0] = w[0];
          r.w[i][1] = w[1];
        }
      } else {
        r.b[i] = *reinterpret_cast<const u32x4_u *>(bytesB + offB[i] + n * ES);
      }
    }
  };
  // load layout -> operand layout through this wave's tiles (LDS instructions of one wave execute in order)
  u32x4 *const tile = lds.stage[wave];
  // WIN: the end of row r's window in segment s, behind the groups: eight bytes (bf16: four), segments of a row exchanged so that the
  // 32 (64) lanes that read at a time fall on different banks
  auto end_of = [&](int r, int s) {
    return reinterpret_cast<uint32_t *>(tile + NG * 128) + Op::WX * (8 * r + (s ^ (BF16 ? 4 * (r >> 3 & 1) : 2 * (r >> 2 & 3))));
  };
  struct Ops {   // what a lane multiplies: its two segments of a row of every group, and (WIN) the ends of the windows
    u32x4 o[NG][2];
    uint32_t w[WIN ? NGB : 1][2][Op::WX];
  };
  auto transpose_all = [&](Ops &x, const Raw &r) {
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) tile[(i / 2) * 128 + (i % 2) * 64 + wslot] = r.a[i];
#pragma unroll
    for (int i = 0; i < NLI; ++i) {
      if constexpr (WIN) {
        tile[(RB + i / 2) * 128 + (i % 2) * 64 + wslot] = r.b[i];
        uint32_t *const e = end_of(8 * i + lr, ls);
        if constexpr (BF16) *e = r.w[i][0];
        else *reinterpret_cast<u32x2 *>(e) = u32x2{r.w[i][0], r.w[i][1]};
      } else if constexpr (CONV) {
        const u32x4 b = r.b[i];
        tile[wslotB[i][0]] = b;
        if constexpr (BF16) {
          tile[wslotB[i][1]] = Op::up(b, r.w[i][0]);
          tile[wslotB[i][2]] = u32x4{b[1], b[2], b[3], r.w[i][0]};
        } else {
          tile[wslotB[i][1]] = u32x4{b[1], b[2], b[3], r.w[i][0]};
          tile[wslotB[i][2]] = u32x4{b[2], b[3], r.w[i][0], r.w[i][1]};
        }
      } else {
        tile[(RB + i / 2) * 128 + (i % 2) * 64 + wslot] = r.b[i];
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      x.o[i][0] = tile[i * 128 + rslot0];
      x.o[i][1] = tile[i * 128 + rslot1];
    }
    if constexpr (WIN)
#pragma unroll
      for (int g = 0; g < NGB; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t *const e = end_of(16 * g + j, q + 4 * h);
          if constexpr (BF16) {
            x.w[g][h][0] = *e;
          } else {
            const u32x2 v = *reinterpret_cast<const u32x2 *>(e);
            x.w[g][h][0] = v[0];
            x.w[g][h][1] = v[1];
          }
        }
    __builtin_amdgcn_wave_barrier();
  };
  f32x4 acc[NB][RB], cor[NB][RB];
  auto clear = [&](f32x4 (&a)[NB][RB]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) a[b][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto mac_all = [&](const Ops &x) {
    typename Op::frag a[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) a[rb] = Op::make(x.o[rb][0], x.o[rb][1]);
    if constexpr (WIN) {
#pragma unroll
      for (int g = 0; g < NGB; ++g) {
        typename Op::frag f[3];
        Op::windows(f, x.o[RB + g], x.w[g]);
#pragma unroll
        for (int d = 0; d < 3; ++d) Op::template mac<RB>(a, f[d], acc[3 * g + d], cor[3 * g + d]);
      }
    } else {
#pragma unroll
      for (int b = 0; b < NB; ++b) Op::template mac<RB>(a, Op::make(x.o[RB + b][0], x.o[RB + b][1]), acc[b], cor[b]);
    }
  };
  // The last, partly empty step: columns at and past N count as zero on both sides.  A lane whose columns are not all there
  // loads the row's last CPL ones (the host takes this kernel for N >= CPL) and moves them down: no load waits for another
  // (column by column, and lane by lane behind branches: 3 us for the one step).
  auto load_ragged = [&](Raw &r, int64_t n) {
    const int64_t own = n + ls * CPL, at = own < p.N - CPL ? own : p.N - CPL, off = at - ls * CPL;
    const int s = own - at < CPL ? int(own - at) : CPL;
    const bool valid = s == 0;
    const bool odd = p.N % CPL != 0;
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) r.a[i] = Op::load_any(bytesA + offA[i] + off * ES);
    if constexpr (!CONV)
#pragma unroll
      for (int i = 0; i < NLI; ++i) r.b[i] = Op::load_any(bytesB + offB[i] + off * ES);
    auto cut = [&](u32x4 &x) {
      if (odd) x = Op::moved(x, s);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = s < CPL ? x[e] : 0u;
    };
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) cut(r.a[i]);
    if constexpr (CONV) {   // (N is a multiple of the group: s is 0 or CPL)
      Raw t;
      load_all(t, 0, pixel(n));
#pragma unroll
      for (int i = 0; i < NLI; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.b[i][e] = valid ? t.b[i][e] : 0u;
#pragma unroll
        for (int e = 0; e < Op::WX; ++e) r.w[i][e] = valid ? t.w[i][e] : 0u;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NLI; ++i) cut(r.b[i]);
    }
  };

  clear(acc);
  if constexpr (!BF16) clear(cor);
  if (steps > 0) {
    // two steps of loads in flight
    Raw raw[2];
#pragma unroll
    for (int d = 0; d < 2; ++d) load_all(raw[d], column(d), at_first[d]);
    auto step = [&](int d, int64_t k) {
      Ops o;
      transpose_all(o, raw[d]);
      const int at = at_next[d];
      at_next[d] = pixel(column(k + 4));
      load_all(raw[d], column(k + 2), at);
      __builtin_amdgcn_sched_barrier(0);   // the loads are on their way before the operands are split and multiplied
      mac_all(o);
    };
    int64_t k = 0;
    for (; k + 1 < steps; k += 2) {
      step(0, k);
      step(1, k + 1);
    }
    if (k < steps) step(0, k);
  }
  if (n_lo + steps * CPI < n_hi) {
    Raw r;
    load_ragged(r, n_lo + steps * CPI);
    Ops o;
    transpose_all(o, r);
    mac_all(o);
  }
  if constexpr (!BF16) {
    float zero = 0.f;   // 0, or NaN where a sum is not finite
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[b][rb][i] = (acc[b][rb][i] + cor[b][rb][i]) * kDown;
          zero = __builtin_fmaf(acc[b][rb][i], 0.f, zero);
        }
    if (__builtin_amdgcn_ballot_w64(zero != 0.f)) {   // (wave-uniform; no barrier inside)
      clear(cor);
      for (int64_t n = n_lo; n < n_hi; n += CPI) {
        Raw r;
        load_ragged(r, n);
        Ops x;
        transpose_all(x, r);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              u32x4 v = x.o[RB + (WIN ? b / 3 : b)][h];
              if constexpr (WIN) {
                const uint32_t (&w)[Op::WX] = x.w[b / 3][h];
                if (b % 3 == 1) v = u32x4{v[1], v[2], v[3], w[0]};
                if (b % 3 == 2) v = u32x4{v[2], v[3], w[0], w[1]};
              }
              Op::mac_fp32(x.o[rb][h], v, cor[b][rb]);
            }
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i)   // (every finite sum stays as it is)
            acc[b][rb][i] = acc[b][rb][i] * 0.f == 0.f ? acc[b][rb][i] : cor[b][rb][i];
    }
  }

  // acc[b][rb][i] = dW block element (row 4 * q + i of row group rb, contraction step 16 * b + j; WIN: tap b % 3 of pixel row
  // 16 * (b / 3) + j); the waves take turns at adding them up
  if constexpr (FAR) find_rows();
  constexpr int TN = (RB * NB + kWaves / 4 - 1) / (kWaves / 4);
  const int first_t = wave / 4;
  float *to[TN];                                // nullptr: nothing to store
#pragma unroll
  for (int x = 0; x < TN; ++x) {
    const int t = first_t + x * (kWaves / 4), b = t % NB;
    // contraction step of this lane's column: 16 * b + j, or (gi) wherever G_i puts stage row 16 * b + j for u_i
    const int st = WIN ? 16 * b0 + 3 * (16 * (b / 3) + j) + b % 3 : 16 * (b0 + b) + j;
    float *const d = RB == 1 || t < NB ? dst[0] : dst[RB - 1];
    const int ui = RB == 1 || t < NB ? dst_ui[0] : dst_ui[RB - 1];
    const bool in = t < RB * NB && d && st < p.nbt * 16;
    const int kk = !in ? -1 : GI ? p.spos[ui * p.nbt * 16 + st] : (st < p.KCR ? st : -1);
    to[x] = kk >= 0 ? d + kk : nullptr;
  }
  __syncthreads();   // (the tiles are done with)
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i) lds.red[wave][(rb * NB + b) * 4 + i][lane] = acc[b][rb][i];
  __syncthreads();
  // wave w: register i = w % 4 of every other (row group, step group)
  float sum[TN];
#pragma unroll
  for (int x = 0; x < TN; ++x) {
    const int e = (first_t + x * (kWaves / 4) < RB * NB ? first_t + x * (kWaves / 4) : 0) * 4 + wave % 4;
    sum[x] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; w += 4)
      sum[x] += (lds.red[w][e][lane] + lds.red[w + 1][e][lane]) + (lds.red[w + 2][e][lane] + lds.red[w + 3][e][lane]);
  }
#pragma unroll
  for (int x = 0; x < TN; ++x)
    if (to[x]) *to[x] = sum[x];
}

template <int RB, bool BF16, bool CONV, bool GI, bool FAR>
rbgp_sddmm_fn pick_nb(int NB) {
  switch (NB) {
    case 1: return sddmm_lines<RB, 1, BF16, CONV, GI, FAR>;
    case 2: return sddmm_lines<RB, 2, BF16, CONV, GI, FAR>;
    case 3: return sddmm_lines<RB, 3, BF16, CONV, GI, FAR>;
  }
  if constexpr (BF16) {
    if constexpr (CONV) {
      if (NB == 6) return sddmm_lines<RB, 6, true, true, GI, FAR>;
    } else {
      if (NB == 4) return sddmm_lines<RB, 4, true, false, GI, false>;
      if (NB == 5) return sddmm_lines<RB, 5, true, false, GI, false>;
    }
  }
  return nullptr;
}
template <bool CONV, bool GI, bool FAR>
rbgp_sddmm_fn find(int RB, int NB, bool bf16) {
  if (RB == 1) return bf16 ? pick_nb<1, true, CONV, GI, FAR>(NB) : pick_nb<1, false, CONV, GI, FAR>(NB);
  if (RB == 2) return bf16 ? pick_nb<2, true, CONV, GI, FAR>(NB) : pick_nb<2, false, CONV, GI, FAR>(NB);
  return nullptr;
}

}  // namespace

rbgp_sddmm_fn rbgp_sddmm_lines_kernel(int RB, int NB, bool bf16, bool conv, bool gi, bool far) {
  if (conv && far) return gi ? find<true, true, true>(RB, NB, bf16) : find<true, false, true>(RB, NB, bf16);
  return conv ? (gi ? find<true, true, false>(RB, NB, bf16) : find<true, false, false>(RB, NB, bf16))
              : (gi ? find<false, true, false>(RB, NB, bf16) : find<false, false, false>(RB, NB, bf16));
}
