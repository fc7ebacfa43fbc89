// The weight gradient's MFMA kernel for most shapes (see rbgp_sddmm.hip for its units): eight waves per workgroup, two per
// SIMD, each with its own range of the batch, RB groups of 16 rows of dO and NB groups of 16 rows of I; a step is 128 bytes
// of a row, one cache line: 32 columns in fp32, 64 in bf16.  Compared with sddmm_reg (steps of 64 bytes, four waves, whole
// stages): twice the bytes in flight, lines asked for once, a unit's outputs split over workgroups before the batch is (no
// partial sums, no second launch), the workgroups of an XCD chosen for the rows they share.
// CONV: the three horizontal taps of a channel row are one window of a lane's columns and one pixel to either side, loaded once
// (16 bytes and 4 or 8 more, aligned to 4 bytes) and written to LDS three times, shifted: a third of the rows of sddmm_reg,
// whose bf16 loads are mostly aligned to 2 bytes.
// fp32: operands are split (rbgp_split.h) after the pass through LDS, and their products go through the bf16 matrix core: 6.5
// vector instructions a value, 36 MFMAs of 16 cycles instead of 48 of 32 for 2 x 3 groups x 32 columns.
//
// us, before (sddmm_reg, with its second launch) -> this kernel: VGG19 conv3 bf16, 8192 columns, fused 19.0 -> 13.7, lowered
// 20.5 -> 15.5, 2368 columns 13.0 -> 8.2; WRN group 1 bf16 fused 27.9 -> 22; conv5 bf16 11.8 -> 10.1, fp32 fused 23.2 -> 20.6;
// VGG19 layer 6 at 1/4 fp32, 2368 columns 19.1 -> 16.3, 320 columns 10.9 -> 6.7; fp32 error against 64-bit sums 1.8e-7 -> 0.8e-7.
// What bounds it (conv5 fp32 fused, timing-only builds): empty loops 5.3 (launch, tables, adding up eight waves), the loads
// alone 11 (lowered 13.4: memory), the passes through LDS alone 12.5, loads and LDS 14.5; the splits keep a wave's issue slot
// (4 to 6 cycles an instruction) busy for 1200 cycles a step.  Tried: twelve waves (23.2, spills), four (25), one step in flight
// (21.1), fp32 MFMAs (22.5), each workgroup's steps starting elsewhere in its range (no change).
#include <hip/hip_runtime.h>

#include "rbgp_sddmm.h"
#include "rbgp_split.h"

using namespace rbgp_split;
using rbgp_sddmm_detail::SddmmParams;

namespace {

constexpr int kWaves = rbgp_sddmm_detail::kLinesWaves;
typedef f32x4 f32x4_u __attribute__((aligned(4)));
typedef bf16x8 bf16x8_u __attribute__((aligned(4)));
typedef bf16x8 bf16x8_any __attribute__((aligned(2)));

template <bool BF16>
struct Operand;
// fp32: the parts of the split operands (rbgp_split.h) go through v_mfma_f32_16x16x32_bf16, the product of the leading
// parts into one accumulator and the five small ones into another; `again` is the fp32 form, for sums that are not finite.
template <>
struct Operand<false> {
  static constexpr int CPL = 4;   // columns per lane and load
  static __device__ __forceinline__ u32x4 load(const void *base, int64_t elem) {
    return __builtin_bit_cast(u32x4, *reinterpret_cast<const f32x4_u *>(static_cast<const float *>(base) + elem));
  }
  static __device__ __forceinline__ u32x4 load_any(const void *base, int64_t elem) { return load(base, elem); }
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
  static __device__ __forceinline__ u32x4 load(const void *base, int64_t elem) {
    return __builtin_bit_cast(u32x4, *reinterpret_cast<const bf16x8_u *>(static_cast<const uint16_t *>(base) + elem));
  }
  static __device__ __forceinline__ u32x4 load_any(const void *base, int64_t elem) {   // (any alignment)
    return __builtin_bit_cast(u32x4, *reinterpret_cast<const bf16x8_any *>(static_cast<const uint16_t *>(base) + elem));
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

// RB: groups of 16 rows of dO per wave; NB: groups of 16 contraction steps per wave.
template <int RB, int NB, bool BF16, bool CONV, bool GI>
__global__ __launch_bounds__(64 * kWaves) void sddmm_lines(SddmmParams p) {
  typedef Operand<BF16> Op;
  constexpr int CPL = Op::CPL, CPI = 8 * CPL;   // columns per lane load / per step: 128 bytes of a row
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int NG = RB + NB;
  // CONV: pixel rows (channel, dy), three taps each, whose windows one step loads: eight per load instruction
  constexpr int NPL = (16 * NB + 23) / 24 < 3 ? (16 * NB + 23) / 24 : 3;   // (a stage has at most 72 steps)
  constexpr int NLI = CONV ? NPL : 2 * NB;      // 16-byte loads of rows of I per step
  constexpr bool kDump = CONV && 24 * NPL > 16 * NB;
  constexpr int kTile = NG * 128 + (kDump ? 64 : 0);   // 16-byte slots of a wave: 16 rows x 128 bytes per group
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
  // Workgroups go to the eight XCDs round-robin in launch order, and each XCD has its own L2: the unit numbers are dealt
  // to the XCDs in eight contiguous runs, so that those of one XCD read few rows (see `order`).
  int x;
  {
    const int total = gridDim.x, xcd = blockIdx.x % 8, each = total / 8, more = total % 8;
    x = xcd * each + (xcd < more ? xcd : more) + int(blockIdx.x) / 8;
  }
  const int piece = x % p.halves; x /= p.halves;
  const int b0 = piece * NB;                    // first 16-step group of this workgroup
  const int g = x % p.RBG; x /= p.RBG;
  const int nu3 = GI ? 1 : p.a3;
  int u3 = 0, sg, v1, part;
  if (p.order == 1) {
    sg = x % p.NSTG; x /= p.NSTG;
    v1 = x % p.c1; x /= p.c1;
    u3 = x % nu3; part = x / nu3;
  } else {
    u3 = x % nu3; x /= nu3;
    sg = x % p.NSTG; x /= p.NSTG;
    v1 = x % p.c1; part = x / p.c1;
  }
  const int RS = 1 << p.lgRS;
  const int32_t *crow = p.colrows + v1 * p.EO, *cpos = p.colpos + v1 * p.EO;
  const int base = v1 * p.tile_rows + sg * p.stage_rows;

  // row r16 of row group rb of this workgroup: (row of dO, or -1; its entry of the tile-row list; its u_i)
  struct RowOf { int64_t row; int entry, ui; };
  auto row_of = [&](int rb, int r16) {
    RowOf o{-1, 0, u3};
    int ri;
    if constexpr (GI) {
      const int rho = (g * RB + rb) * 16 + r16;
      ri = rho % p.R;
      o.ui = (rho / p.R) % p.a3;
      o.entry = rho / (p.R * p.a3);
    } else {
      o.entry = (g * RB + rb) * p.MG + (r16 >> p.lgRS);
      ri = r16 & (RS - 1);
    }
    if (o.entry < p.EO && ri < p.R)
      o.row = ((int64_t(crow[o.entry]) * p.a2 + ri / p.a4) * p.a3 + o.ui) * p.a4 + ri % p.a4;
    return o;
  };
  int64_t offA[2 * RB];   // element offset of this lane's 16 bytes in step 0
#pragma unroll
  for (int i = 0; i < 2 * RB; ++i) {
    const int64_t row = row_of(i / 2, lr + 8 * (i % 2)).row;
    offA[i] = (row < 0 ? 0 : row) * p.ld_dO + ls * CPL;
  }
  int64_t offB[NLI];      // CONV: byte offset of the row's window inside X (below 2 GiB)
  int wslotB[CONV ? NPL : 1][3];
  if constexpr (CONV) {
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int kk = 48 * (b0 / 3) + 3 * (8 * i + lr);     // first tap of the pair (b0 is a multiple of 3)
      const int sr = GI ? (kk < p.src_rows ? kk : 0) : (kk < p.KCR ? p.rowtab[u3 * p.nbt * 16 + kk] : 0);
      const int k = base + sr;                             // channel k / 9, dy = (k % 9) / 3 - 1, dx = -1
      offB[i] = (int64_t(k / 9) * p.chan_elems + ((k % 9) / 3 - 1) * p.conv_w2 - 1) * ES;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int row = 3 * (8 * i + lr) + d;
        wslotB[i][d] = row < 16 * NB ? (RB + row / 16) * 128 + (row % 16) * 8 + (ls ^ (row & 7)) : NG * 128 + lane;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NLI; ++i) {   // padding steps read row 0 of the stage
      const int b = b0 + i / 2, r = lr + 8 * (i % 2), sr = 16 * b + r;
      const int k = base + (GI ? (sr < p.src_rows ? sr : 0) : (b < p.nbt ? p.rowtab[(u3 * p.nbt + b) * 16 + r] : 0));
      offB[i] = int64_t(k) * p.ldI + ls * CPL;
    }
  }
  // CONV: where this lane's group of columns starts inside a channel (columns are pixels in image order)
  auto pixel = [&](int64_t n) { return CONV ? p.colbase[n / CPL + ls] * ES : 0; };
  __amdgpu_buffer_rsrc_t xrsrc;
  if constexpr (CONV) xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.I), 0, int(p.x_bytes), 0x00020000);

  // What one step has in flight.  CONV: the window of CPL + 2 pixels that the three horizontal taps of a lane's columns share.
  struct Raw {
    u32x4 a[2 * RB], b[NLI];
    uint32_t w[CONV ? NPL : 1][2];
  };
  // (`at`: pixel(n), looked up by the caller -- ahead of time inside the loop, where a lookup right before its use
  // would have to wait for every load in flight)
  auto load_all = [&](Raw &r, int64_t n, int at) {
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) r.a[i] = Op::load(p.dO, offA[i] + n);
#pragma unroll
    for (int i = 0; i < NLI; ++i) {
      if constexpr (CONV) {
        const int o = int(offB[i]) + at;
        r.b[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, o, 0, 0);
        if constexpr (BF16) {
          r.w[i][0] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, o, 16, 0);
        } else {
          const auto w = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, o, 16, 0);
          r.w[i][0] = w[0];
          r.w[i][1] = w[1];
        }
      } else {
        r.b[i] = Op::load(p.I, offB[i] + n);
      }
    }
  };
  // load layout -> operand layout through this wave's tiles (LDS instructions of one wave execute in order)
  u32x4 *const tile = lds.stage[wave];
  auto transpose_all = [&](u32x4 (&o)[NG][2], const Raw &r) {
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) tile[(i / 2) * 128 + (i % 2) * 64 + wslot] = r.a[i];
#pragma unroll
    for (int i = 0; i < NLI; ++i) {
      if constexpr (CONV) {
        const u32x4 b = r.b[i];
        const uint32_t w0 = r.w[i][0], w1 = r.w[i][1];
        tile[wslotB[i][0]] = b;
        if constexpr (BF16) {
          tile[wslotB[i][1]] = u32x4{__builtin_amdgcn_alignbit(b[1], b[0], 16), __builtin_amdgcn_alignbit(b[2], b[1], 16),
                                     __builtin_amdgcn_alignbit(b[3], b[2], 16), __builtin_amdgcn_alignbit(w0, b[3], 16)};
          tile[wslotB[i][2]] = u32x4{b[1], b[2], b[3], w0};
        } else {
          tile[wslotB[i][1]] = u32x4{b[1], b[2], b[3], w0};
          tile[wslotB[i][2]] = u32x4{b[2], b[3], w0, w1};
        }
      } else {
        tile[(RB + i / 2) * 128 + (i % 2) * 64 + wslot] = r.b[i];
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      o[i][0] = tile[i * 128 + rslot0];
      o[i][1] = tile[i * 128 + rslot1];
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
  auto mac_all = [&](const u32x4 (&o)[NG][2]) {
    typename Op::frag a[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) a[rb] = Op::make(o[rb][0], o[rb][1]);
#pragma unroll
    for (int b = 0; b < NB; ++b) Op::template mac<RB>(a, Op::make(o[RB + b][0], o[RB + b][1]), acc[b], cor[b]);
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
    for (int i = 0; i < 2 * RB; ++i) r.a[i] = Op::load_any(p.dO, offA[i] + off);
    if constexpr (!CONV)
#pragma unroll
      for (int i = 0; i < NLI; ++i) r.b[i] = Op::load_any(p.I, offB[i] + off);
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
        r.w[i][0] = valid ? t.w[i][0] : 0u;
        if constexpr (!BF16) r.w[i][1] = valid ? t.w[i][1] : 0u;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NLI; ++i) cut(r.b[i]);
    }
  };

  const int64_t n_lo = (int64_t(part) * kWaves + wave) * p.chunk;
  const int64_t n_hi = n_lo + p.chunk < p.N ? n_lo + p.chunk : p.N;   // (n_lo may lie past N: empty range)
  const int64_t steps = n_hi > n_lo ? (n_hi - n_lo) / CPI : 0;        // whole steps
  clear(acc);
  if constexpr (!BF16) clear(cor);
  if (steps > 0) {
    // two steps of loads in flight; past the last step the loads repeat it (in bounds)
    const int64_t n_last = n_lo + (steps - 1) * CPI;
    auto column = [&](int64_t k) {
      const int64_t c = n_lo + k * CPI;
      return c < n_last ? c : n_last;
    };
    Raw raw[2];
    int at_next[2];   // pixel(column(k + 2)) of the step that refills set d next, requested one round earlier
#pragma unroll
    for (int d = 0; d < 2; ++d) load_all(raw[d], column(d), pixel(column(d)));
#pragma unroll
    for (int d = 0; d < 2; ++d) at_next[d] = pixel(column(2 + d));
    auto step = [&](int d, int64_t k) {
      u32x4 o[NG][2];
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
    u32x4 o[NG][2];
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
        u32x4 o[NG][2];
        transpose_all(o, r);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) Op::mac_fp32(o[rb][h], o[RB + b][h], cor[b][rb]);
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

  // acc[b][rb][i] = dW block element (row 4 * q + i of row group rb, contraction step 16 * b + j); the waves take turns
  // at adding them up
  __syncthreads();   // (the tiles are done with)
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i) lds.red[wave][(rb * NB + b) * 4 + i][lane] = acc[b][rb][i];
  __syncthreads();
  // wave w: register i = w % 4 of every other (row group, step group)
#pragma unroll
  for (int t = 0; t < RB * NB; ++t) {
    if (t % (kWaves / 4) != wave / 4) continue;
    const int rb = t / NB, b = t % NB, e = t * 4 + wave % 4;
    const RowOf o = row_of(rb, 4 * q + wave % 4);
    if (o.row < 0) continue;
    // the stage is fragment cpos * NSTG + sg of the row: KCR consecutive kept values
    float *dst = p.out + int64_t(part) * p.nnz + o.row * p.rowdeg + int64_t(cpos[o.entry] * p.NSTG + sg) * p.KCR;
    // contraction step of this lane's column: 16 * b + j, or (gi) wherever G_i puts stage row 16 * b + j for u_i
    const int st = 16 * (b0 + b) + j;
    const int kk = b0 + b >= p.nbt ? -1 : GI ? p.spos[o.ui * p.nbt * 16 + st] : (st < p.KCR ? st : -1);
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; w += 4)
      sum += (lds.red[w][e][lane] + lds.red[w + 1][e][lane]) + (lds.red[w + 2][e][lane] + lds.red[w + 3][e][lane]);
    if (kk >= 0) dst[kk] = sum;
  }
}

template <int RB, bool BF16, bool CONV, bool GI>
rbgp_sddmm_fn pick_nb(int NB) {
  switch (NB) {
    case 1: return sddmm_lines<RB, 1, BF16, CONV, GI>;
    case 2: return sddmm_lines<RB, 2, BF16, CONV, GI>;
    case 3: return sddmm_lines<RB, 3, BF16, CONV, GI>;
  }
  if constexpr (BF16) {
    if (NB == 4) return sddmm_lines<RB, 4, true, CONV, GI>;
    if (NB == 5) return sddmm_lines<RB, 5, true, CONV, GI>;
  }
  return nullptr;
}
template <bool CONV, bool GI>
rbgp_sddmm_fn find(int RB, int NB, bool bf16) {
  if (RB == 1) return bf16 ? pick_nb<1, true, CONV, GI>(NB) : pick_nb<1, false, CONV, GI>(NB);
  if (RB == 2) return bf16 ? pick_nb<2, true, CONV, GI>(NB) : pick_nb<2, false, CONV, GI>(NB);
  return nullptr;
}

}  // namespace

rbgp_sddmm_fn rbgp_sddmm_lines_kernel(int RB, int NB, bool bf16, bool conv, bool gi) {
  return conv ? (gi ? find<true, true>(RB, NB, bf16) : find<true, false>(RB, NB, bf16))
              : (gi ? find<false, true>(RB, NB, bf16) : find<false, false>(RB, NB, bf16));
}
