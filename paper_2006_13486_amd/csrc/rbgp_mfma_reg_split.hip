// fp32 product of the register-streaming family on the bf16 matrix core: every fp32 operand is split into three
// bf16 numbers (8 + 8 + 8 mantissa bits: x = x0 + x1 + x2 exactly) and the six products that reach fp32 accuracy --
// x0y0, x0y1, x1y0, x1y1, x0y2, x2y0; the rest is at most about 2^-24 of |xy|, an fp32 rounding, as |x1| <= 2^-8 |x|
// and |x2| <= 2^-17 |x| -- go through v_mfma_f32_32x32x16_bf16, which multiplies 16 times as many operands per cycle
// as the fp32 forms: 2.7 times fewer matrix-core cycles for the six of them.
//
// For masks whose 16-row MFMA groups come in pairs with one stage list (rows of G_r moved into the tile-row index:
// filled masks, merged columns, layers at density 1/2).  A wave owns 32 rows (two tile rows), one G_i vertex and 128
// columns, and walks the same stages of the same packed fp32 weights as spmm_reg, 16 contraction steps at a time.
// Operand layout: lane l holds, of row (column) l % 32, the eight steps 16 q + 4 w + 2 (l / 32) + gg (w = 0..3,
// gg = 0, 1) of block q of a stage -- two 16-byte pieces of a packed fragment for the weights, eight rows of I with
// four columns each (16-byte loads, 512 contiguous bytes per row) for the four 32-column blocks t, which
// hold the columns 4 j + t: the split pairs values of two rows in one conversion, so no transpose is needed, and the
// accumulators of the four blocks are four consecutive columns of O again.
//
// Precision.  x0y0 accumulates by itself; the five small products have accumulators of their own, added once at the
// end.  Then an output sees one rounding at its full magnitude per 16 steps (the fp32 forms: one per step, on four
// partial sums).  Against 64-bit sums, 2-norm, random operands of 1024 steps: 1.8e-7, four-block fp32 form 2.9e-7
// (one accumulator for all six: 4.9e-7).  Scaling by 2^23 (kUp) keeps every part of every operand a normal bf16 number.
// An operand that is Inf, NaN or at least 2^105 makes Inf - Inf of the split, and sums from 2^82 on leave fp32's range: a
// wave that finds a non-finite sum multiplies its tile again with fp32 MFMAs, which keep Inf as Inf.
//
// What bounds it: per 16 steps x 32 rows x 128 columns a wave issues 24 MFMAs (768 cycles) and 275 vector
// instructions, most of them the splits (1100 cycles; the scaling is 40 of them and costs 1-5 %); two waves share a SIMD, one
// multiplying while the other splits.  Measured, 4096^3 fp32, one row per column set at density 1/8 (34.4 GFLOP on the
// filled mask): 309 us on the fp32 MFMAs -> 212.
#include <hip/hip_runtime.h>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"
#include "rbgp_split.h"

using namespace rbgp_reg;
using namespace rbgp_split;

namespace {

typedef f32x4 f32x4_u __attribute__((aligned(4)));
typedef uint16_t halfword __attribute__((may_alias));   // (LDS written by halfwords and read as operands)

// A stage is walked in p.nq blocks of 16 contraction steps (the last one may be padding in part: zero weights).
__global__ __launch_bounds__(256, 2) void spmm_reg_split(RegParams p) {
  constexpr int CW = 128;                       // columns per wave
  constexpr int QB = 4 * 16 * 16;               // bytes of 16 steps of a packed fragment (16 rows)
  extern __shared__ __attribute__((aligned(16))) unsigned char red[];   // partial sums of a split stage list
  __shared__ __attribute__((aligned(16))) int rowoff[5 * 16];           // [q][lane / 32][e]: byte offset of a step's row of I
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int lgS = p.lgS, S = 1 << lgS;
  const int ks = wid & (S - 1);
  table_args(p);
  WgCoord wg;
  if (!wg_coord(p, &wg)) return;                // (the whole workgroup)
  const int u1 = wg.cl * 2, u3 = wg.u3;         // first of the wave's two tile rows
  const int nt = (wg.ntq << (2 - lgS)) + (wid >> lgS);
  const bool valid = nt < p.ntiles;
  const int64_t n0 = int64_t(nt) * CW;
  const uint32_t n0b = p.conv ? 0u : uint32_t(nt) * uint32_t(CW * 4);
  const int h = lane >> 5, j = lane & 31;

  const int nq = p.nq;
  if (int(threadIdx.x) < nq * 16) {
    const int q = threadIdx.x >> 4, hh = (threadIdx.x >> 3) & 1, e = threadIdx.x & 7;
    const int kk = 16 * q + 4 * (e & 3) + 2 * hh + (e >> 2);
    const int r = kk < p.kcr ? p.rowtab[u3 * p.no4 + kk] : 0;
    // (< 2^31: checked by the host; padding steps lie past every extent and read zeros without a memory access)
    rowoff[threadIdx.x] = kk >= p.kcr ? int(0x80000000u) : p.conv ? r : r * (int(p.ldI) * 4);
  }
  // the wave's own stages, one per lane (see spmm_reg); both tile rows have the same list and the same positions
  const int TS = p.tstride;
  const int own = ks + (lane << lgS);
  const int32_t *stg = p.stages + int64_t(u1) * 2 * TS + (own < TS ? own : TS - 1);
  const int tb = stg[0], tf = stg[TS];
  const int cnt0 = p.counts[u1];
  const int cnt = __builtin_amdgcn_readfirstlane(valid && cnt0 > ks ? (cnt0 - ks + S - 1) >> lgS : 0);
  const int rov = p.rowofs[lane & 15];
  const int col = p.conv ? p.colbase[valid ? int(n0 >> 2) + j : 0] & ~3 : j * 16;   // the lane's four columns
  const int fstr = p.fpm * p.a3 * p.frag_bytes;   // from one tile row's weights to the next one's
  const int alane = (j >> 4) * fstr + ((2 * h) * 16 + (j & 15)) * 16;
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  const int tbu = p.conv ? int(uint32_t(tb < 0 ? 0 : tb) / 9u) : (tb < 0 ? 0 : tb);
  const uint64_t i_first = reinterpret_cast<uint64_t>(p.I) + uint64_t(uint32_t(tbu)) * p.row_bytes + n0b;
  const int ib_lo = int(uint32_t(i_first)), ib_hi = int(uint32_t(i_first >> 32));
  // (to the last column of the stage's last row, so that an extent stays below 2^31: SRC rows of ldI do, checked by the host)
  const int rows_left = p.last_row - tbu < p.src_rows - 1 ? p.last_row - tbu : p.src_rows - 1;
  const int ib_ext = (tb >= 0 && valid) ? int(uint32_t(rows_left) * p.row_bytes + (p.n_bytes - n0b)) : 0;
  const int aoff = tf >= 0 ? ((u1 * p.fpm + tf) * p.a3 + u3) * p.frag_bytes : kOob;
  float *const out = p.O;
  const int64_t out_ld = p.ldO, out_n = p.N;
  const int out_tm = p.tm, out_a4 = p.a4, out_r = p.R;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (!valid && lgS == 0) return;

  f32x4 B[8], A[2];
  // the loads of block q of stage s (past the wave's count: zero extent, weights past the end of the buffer)
  auto load = [&](int s, int q) {
    const int tl = s < 63 ? s : 63;
    const bool live = s < cnt;
    const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_lo, tl))) |
                          (uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_hi, tl))) << 32);
    const int ext = __builtin_amdgcn_readlane(ib_ext, tl), av = __builtin_amdgcn_readlane(aoff, tl);
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, live ? ext : 0, kRsrcFlags);
    const int4 *ro = reinterpret_cast<const int4 *>(rowoff + q * 16 + h * 8);
    const int4 r0 = ro[0], r1 = ro[1];
    const int off[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) B[e] = load_x4(rb, off[e] + col, 0);
#pragma unroll
    for (int gg = 0; gg < 2; ++gg) A[gg] = load_x4(rw, (live ? av : kOob) + alane + gg * 256, q * QB);
  };

  f32x16 acc[4], cor[4];
  auto clear = [&](f32x16 (&x)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) x[t][i] = 0.f;
  };
  clear(acc);
  clear(cor);
  load(0, 0);
  {
    int s = 0, q = 0;
    for (const int blocks = cnt * nq; blocks > s * nq + q;) {
      Split b[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float x[8] = {B[0][t], B[1][t], B[2][t], B[3][t], B[4][t], B[5][t], B[6][t], B[7][t]};
        b[t] = split8(x);
      }
      const float w[8] = {A[0][0], A[0][1], A[0][2], A[0][3], A[1][0], A[1][1], A[1][2], A[1][3]};
      const Split a = split8(w);
      q = q + 1 < nq ? q + 1 : 0;
      s += q == 0;
      load(s, q);
      __builtin_amdgcn_sched_barrier(0);   // the next block's loads are on their way before the MFMAs start
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b[t].p[0], acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) cor[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b[t].p[1], cor[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) cor[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[1], b[t].p[0], cor[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) cor[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[1], b[t].p[1], cor[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) cor[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b[t].p[2], cor[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) cor[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[2], b[t].p[0], cor[t], 0, 0, 0);
    }
  }
  bool again = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) again |= add_up(acc[t], cor[t]) && n0 + j * 4 + t < out_n;
  if (__builtin_amdgcn_ballot_w64(again)) {   // (wave-uniform; no barrier inside)
    clear(cor);
    for (int s = 0; s < cnt; ++s)
      for (int q = 0; q < nq; ++q) {
        load(s, q);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            cor[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[e / 4][e % 4], B[e][t], cor[t], 0, 0, 0);
      }
#pragma unroll
    for (int t = 0; t < 4; ++t) take_not_finite(acc[t], cor[t]);
  }

  // Epilogue.  Unit i = register i of the four accumulators: weight row 8 (i / 4) + 4 (lane / 32) + i % 4 of the wave's
  // 32, the lane's four columns 4 j .. 4 j + 3.
  const bool whole = n0 + j * 4 + 4 <= out_n;
  auto store_unit = [&](int i, f32x4 v) {
    const int r32 = 8 * (i / 4) + 4 * h + i % 4, r = r32 & 15;
    const int ro = __builtin_amdgcn_ds_bpermute(r * 4, rov);
    if (valid && r < out_r) {
      const int64_t m = int64_t(u1 + (r32 >> 4)) * out_tm + u3 * out_a4 + ro;
      float *o = out + m * out_ld + n0 + j * 4;
      if (whole) {
        store_x4(o, v);
      } else {
#pragma unroll
        for (int w = 0; w < 4; ++w)
          if (n0 + j * 4 + w < out_n) o[w] = v[w];
      }
    }
  };
  auto unit = [&](int i) { return f32x4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]}; };
  if (lgS == 0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) store_unit(i, unit(i));
  } else {
    // as in spmm_reg: a wave leaves the units it does not own in LDS and adds up the ones it owns in wave order
    f32x4 *const red4 = reinterpret_cast<f32x4 *>(red);
    const int per_wave = (16 >> lgS) * (S - 1);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int o = i & (S - 1);
      if (o != ks) red4[(wid * per_wave + (i >> lgS) * (S - 1) + o - (o > ks ? 1 : 0)) * 64 + lane] = unit(i);
    }
    __syncthreads();
    const int w0 = wid & ~(S - 1);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if ((i & (S - 1)) == ks) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        for (int kk = 0; kk < S; ++kk) {
          if (kk == ks)
            v += unit(i);
          else
            v += red4[((w0 + kk) * per_wave + (i >> lgS) * (S - 1) + ks - (ks > kk ? 1 : 0)) * 64 + lane];
        }
        store_unit(i, v);
      }
    }
  }
}

// The same product where four pairs of tile rows have one stage list: the four waves of a workgroup take one pair each
// on the same 128 columns, split every value of I once between them and pass the parts through LDS (stored in the
// operand layout, 16 bytes per lane: no bank conflicts).  Vector instructions per MFMA fall from 11 to 5, which leaves
// the matrix core as the bound (58 % busy at the 1.7-1.9 GHz the card clocks down to under this load: 1.2 PFLOP/s of bf16
// products, what a large library product in bf16 reaches); one barrier per two blocks of 16 steps, double-buffered.
// 4096^3 fp32, one row per column set at density 1/4 (68.7 GFLOP on the filled mask): 519 us on the fp32 MFMAs -> 330
// (waves by themselves 409; two waves sharing 64 columns 415, four sharing 64 columns 379).
// A lane holds one column of a 32-column block.
//
// SPARSE: filled masks whose rows keep at most one of the steps k and k + 16 of a 32-step stage (a 2-lift puts an edge on
// one of two vertices half of G_i apart, never on both).  v_smfmac_f32_32x32x32_bf16 multiplies two weights of every four
// steps by the rows of I that its index operand names, so the zeros that fill G_i in are not multiplied: half of the
// MFMAs, each about 1.3 times as long (in bf16 products 3.8 against 2.4 PFLOP/s on registers).  The two blocks of weights of
// a stage become one (bit by bit or, one of the two is +0), which is split once; places are the same in every stage and
// are held in a register.  Operands: the lane of half h holds the compressed weights of steps 4 w + 2 h + g (w = 0..3, then
// g = 0, 1), and the first four belong to the rows of I in the lanes of half 0, the others to half 1, so there the lane of
// half h holds the rows of steps 4 w + h, then 4 w + 2 + h, each with its partner 16 further.
// 4096^3 fp32, one row per column set at density 1/4: 330 -> 247 us, error against 64-bit sums 1.53e-7 -> 1.43e-7 (half as
// many roundings); bound by issue: a stage's 24 MFMAs and 198 vector instructions per wave keep the matrix core busy for 40 %
// and the vector units for 50 % of the launch, at 1.8 GHz, and waves wait for 14 % of theirs (waves of 64 rows x 64 columns, which
// read half as much LDS and split the weights twice: 263 against 238 on one machine).
template <bool SPARSE>
__global__ __launch_bounds__(256, 2) void spmm_reg_split_shared(RegParams p) {
  constexpr int NT = 4, CW = NT * 32;           // 32-column blocks, columns of a workgroup
  __shared__ __attribute__((aligned(16))) u32x4 parts[2][2][NT][3][64];
  __shared__ __attribute__((aligned(16))) int rowoff[SPARSE ? 2 : 1][5 * 16];   // [order of the steps][q][lane / 32][e]
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  table_args(p);
  WgCoord wg;
  if (!wg_coord(p, &wg)) return;
  const int u1 = wg.cl * 8 + 2 * wid, u3 = wg.u3;
  const int nt = wg.ntq;
  const int64_t n0 = int64_t(nt) * CW;
  const uint32_t n0b = p.conv ? 0u : uint32_t(nt) * uint32_t(CW * 4);
  const int h = lane >> 5, j = lane & 31;
  const int nq = p.nq;
  if (int(threadIdx.x) < nq * 16) {
    const int q = threadIdx.x >> 4, hh = (threadIdx.x >> 3) & 1, e = threadIdx.x & 7;
    const int kk = 16 * q + 4 * (e & 3) + 2 * hh + (e >> 2);
    const int r = kk < p.kcr ? p.rowtab[u3 * p.no4 + kk] : 0;
    // (< 2^31: checked by the host; padding steps lie past every extent and read zeros without a memory access)
    rowoff[0][threadIdx.x] = kk >= p.kcr ? int(0x80000000u) : p.conv ? r : r * (int(p.ldI) * 4);
    if constexpr (SPARSE) {                     // (32 steps, all of them rows of I)
      const int ks = 16 * q + 4 * (e & 3) + hh + 2 * (e >> 2);
      rowoff[1][threadIdx.x] = p.rowtab[u3 * p.no4 + ks] * (int(p.ldI) * 4);
    }
  }
  const int TS = p.tstride;
  const int32_t *stg = p.stages + int64_t(u1) * 2 * TS + lane;   // one stage per lane (at most 64: checked by the host)
  const int tb = stg[0], tf = stg[TS];
  const int cnt = __builtin_amdgcn_readfirstlane(p.counts[u1]);
  const int rov = p.rowofs[lane & 15];
  const int which = SPARSE ? p.pairs[((u1 + (j >> 4)) % p.fold * 2 + h) * 16 + (j & 15)] : 0;
  int col[NT];                                  // byte offset of the lane's column of every block
#pragma unroll
  for (int t = 0; t < NT; ++t)
    col[t] = p.conv ? (p.colbase[int((n0 + 32 * t + j) >> 2)] & ~3) + (j & 3) * 4 : (32 * t + j) * 4;
  const int fstr = p.fpm * p.a3 * p.frag_bytes;
  const int alane = (j >> 4) * fstr + ((2 * h) * 16 + (j & 15)) * 16;
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  const int tbu = p.conv ? int(uint32_t(tb < 0 ? 0 : tb) / 9u) : (tb < 0 ? 0 : tb);
  const uint64_t i_first = reinterpret_cast<uint64_t>(p.I) + uint64_t(uint32_t(tbu)) * p.row_bytes + n0b;
  const int ib_lo = int(uint32_t(i_first)), ib_hi = int(uint32_t(i_first >> 32));
  // (to the last column of the stage's last row, so that an extent stays below 2^31: SRC rows of ldI do, checked by the host)
  const int rows_left = p.last_row - tbu < p.src_rows - 1 ? p.last_row - tbu : p.src_rows - 1;
  const int ib_ext = tb >= 0 ? int(uint32_t(rows_left) * p.row_bytes + (p.n_bytes - n0b)) : 0;
  const int aoff = tf >= 0 ? ((u1 * p.fpm + tf) * p.a3 + u3) * p.frag_bytes : kOob;
  float *const out = p.O;
  const int64_t out_ld = p.ldO, out_n = p.N;
  const int out_tm = p.tm, out_a4 = p.a4, out_r = p.R;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  auto stage_rsrc = [&](int s) {
    const int tl = s < 63 ? s : 63;
    const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_lo, tl))) |
                          (uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_hi, tl))) << 32);
    const int ext = __builtin_amdgcn_readlane(ib_ext, tl);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, s < cnt ? ext : 0, kRsrcFlags);
  };
  auto load_b = [&](float (&x)[8], int s, int q, int c, int order) {
    const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
    const int4 *ro = reinterpret_cast<const int4 *>(rowoff[order] + q * 16 + h * 8);
    const int4 r0 = ro[0], r1 = ro[1];
    const int off[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, off[e] + c, 0, 0));
  };
  auto load_a = [&](f32x4 (&x)[2], int s, int q) {
    const int av = __builtin_amdgcn_readlane(aoff, s < 63 ? s : 63);
#pragma unroll
    for (int gg = 0; gg < 2; ++gg) x[gg] = load_x4(rw, (s < cnt ? av : kOob) + alane + gg * 256, q * 1024);
  };
  float braw[2][8];                             // the wave splits column block `wid` of both blocks of steps of a round
  f32x4 araw[2][2];
  const int own_col = wid == 0 ? col[0] : wid == 1 ? col[1] : wid == 2 ? col[2] : col[3];
  int s0 = 0, q0 = 0;                           // the block of steps whose loads are issued next
  auto load_round = [&]() {
    const int q1 = q0 + 1 < nq ? q0 + 1 : 0, s1 = s0 + (q1 == 0);
    load_a(araw[0], s0, q0);
    load_a(araw[1], s1, q1);
    load_b(braw[0], s0, q0, own_col, SPARSE);
    load_b(braw[1], s1, q1, own_col, SPARSE);
    q0 = q1 + 1 < nq ? q1 + 1 : 0;
    s0 = s1 + (q0 == 0);
  };

  f32x16 acc[NT], cor[NT];
  auto clear = [&](f32x16 (&x)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) x[t][i] = 0.f;
  };
  clear(acc);
  clear(cor);
  load_round();
  const int rounds = (cnt * nq + 1) / 2;
  for (int r = 0; r < rounds; ++r) {
    const int buf = r & 1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      Split b;
      if constexpr (SPARSE) {                   // groups of four: the rows of steps k, k + 16, k + 4, k + 20
        const float x[8] = {braw[0][4 * u], braw[1][4 * u], braw[0][4 * u + 1], braw[1][4 * u + 1],
                            braw[0][4 * u + 2], braw[1][4 * u + 2], braw[0][4 * u + 3], braw[1][4 * u + 3]};
        b = split8(x);
      } else {
        b = split8(braw[u]);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) parts[buf][u][wid][k][lane] = __builtin_bit_cast(u32x4, b.p[k]);
    }
    Split a[2];
    if constexpr (SPARSE) {                     // (one of the two is +0)
      float w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = __uint_as_float(__float_as_uint(araw[0][e / 4][e % 4]) | __float_as_uint(araw[1][e / 4][e % 4]));
      a[0] = split8(w);
    }
#pragma unroll
    for (int u = 0; u < (SPARSE ? 0 : 2); ++u) {
      const float w[8] = {araw[u][0][0], araw[u][0][1], araw[u][0][2], araw[u][0][3],
                          araw[u][1][0], araw[u][1][1], araw[u][1][2], araw[u][1][3]};
      a[u] = split8(w);
    }
    load_round();                               // (past the end: sentinels, no memory access)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
    if constexpr (SPARSE) {
#pragma unroll
      for (int t = 0; t < NT; t += 2) {
        bf16x16 b[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 3; ++k)
            b[x][k] = joined(parts[buf][0][t + x][k][lane], parts[buf][1][t + x][k][lane]);
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            f32x16 &d = k == 0 ? acc[t + x] : cor[t + x];
            d = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a[0].p[pa[k]], b[x][pb[k]], d, which, 0, 0);
          }
      }
    }
#pragma unroll
    for (int u = 0; u < (SPARSE ? 0 : 2); ++u)
#pragma unroll
      for (int t = 0; t < NT; t += 2) {
        bf16x8 b[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 3; ++k) b[x][k] = __builtin_bit_cast(bf16x8, parts[buf][u][t + x][k][lane]);
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            f32x16 &d = k == 0 ? acc[t + x] : cor[t + x];
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u].p[pa[k]], b[x][pb[k]], d, 0, 0, 0);
          }
      }
  }
  bool again = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) again |= add_up(acc[t], cor[t]) && n0 + 32 * t + j < out_n;
  if (__builtin_amdgcn_ballot_w64(again)) {   // (wave-uniform; no barrier inside)
    clear(cor);
    for (int s = 0; s < cnt; ++s)
      for (int q = 0; q < nq; ++q) {
        load_a(araw[0], s, q);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float x[8];
          load_b(x, s, q, col[t], 0);
#pragma unroll
          for (int e = 0; e < 8; ++e) cor[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(araw[0][e / 4][e % 4], x[e], cor[t], 0, 0, 0);
        }
      }
#pragma unroll
    for (int t = 0; t < 4; ++t) take_not_finite(acc[t], cor[t]);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r32 = 8 * (i / 4) + 4 * h + i % 4, r = r32 & 15;
    const int ro = __builtin_amdgcn_ds_bpermute(r * 4, rov);
    if (r < out_r) {
      float *o = out + (int64_t(u1 + (r32 >> 4)) * out_tm + u3 * out_a4 + ro) * out_ld + n0 + j;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (n0 + 32 * t + j < out_n) __builtin_nontemporal_store(acc[t][i], o + 32 * t);
    }
  }
}

// The LDS family's product (RBGP_KERNEL_MFMA, fp32) on the bf16 matrix core, for masks whose G_o and G_i are both sparse:
// a tile of G_o with four rows per column set and |G_i.V| |G_b.V| = 32 columns is multiplied as a dense 32-step block, the
// structural zeros of G_i included (at most three in four), because a 32x32x16 bf16 MFMA does 16 times the products of
// the 4x4x1 fp32 form per cycle.  Workgroup: 128 rows of a tile row (32 G_i vertices, a wave eight of them) x 32 NT columns; with KSP =
// 2, two such groups of four waves take every other stage and add their sums through LDS.  A stage's kept weights (one 16-byte load per lane holds four rows of one step; two for KS = 16) are split and
// scattered to their steps in a wave-private LDS block whose other entries stay zero: the pattern of G_i is the same in
// every tile.  I as in spmm_reg_split_shared, a round being one stage.  One Inf in I makes every sum of its
// column in the tile rows with that tile non-finite (the zeros of G_i are multiplied): such sums are added up again from
// the kept weights, with the 4x4x1 MFMAs and in the order of spmm_mfma.  4096 x 4096, G_o and G_i at 1/4, N = 1531:
// 126 -> 83 us, error against 64-bit sums 2.0e-7 -> 7.6e-8, with the sparse MFMA (SPARSE, see spmm_reg_split_shared: no
// vertex keeps both k and k + 16; the weights are scattered among the 16 steps) 65 and 7.4e-8; inputs with one infinity 1.34 times
// that, with no finite column 1.49 times (dense, a lane adding its sums up one by one: 3.7 and 11 times).
// What bounds it: a stage's chain (split, LDS, barrier, LDS, 24 products of two accumulators each) with 1.5 waves a SIMD, 128 columns:
// 64 columns a workgroup need half of the registers and 37 KB of LDS, three run on a CU: 65 -> 56 us.  Vector instructions (half of them
// splits) and products, one after the other on a SIMD, are then 49 k and 37 k of its 114 k cycles at 2.07 GHz.  The rows of a wave's weights in different banks (row_to; a scattered write met four others):
// bank conflicts 7.1 M -> 2.4 M cycles, 57.5 -> 55 us, one column 24 -> 22.7.  Tried there: two stages of
// loads in flight 57; the next stage split beside the products of this one 63 (the loads are waited for earlier); four groups of
// waves on few columns 24-28 (spills) against 23-25 with two; weights through LDS as loaded, split in operand layout with their zeros
// (fewer LDS instructions, a quarter more vector ones) 59.
template <int KS, bool SPARSE, int NT, int KSP>
__global__ __launch_bounds__(256 * KSP, KSP == 1 && NT == 2 ? 3 : 2) void spmm_mfma_split(SplitTileParams p) {
  constexpr int CW = 32 * NT, IT = KS / 8;
  constexpr int TU = NT / 2;                    // blocks of 16 steps that a wave splits, of one column block
  struct Stage {                                // of the waves that take every KSP-th stage
    u32x4 parts[2][2][NT][3][64];
  };
  constexpr int WB = SPARSE ? 1 : 2;            // blocks of operands that hold a stage's weights
  __shared__ __attribute__((aligned(16))) union {
    Stage stage[KSP];
    float red[KSP > 1 ? KSP - 1 : 1][KSP > 1 ? NT : 1][16][4][64];   // sums of the others
  } lds;
  __shared__ __attribute__((aligned(16))) u32x4 wparts[4 * KSP][3][WB][64];  // [wave][part][16 steps][operand lane]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), wid = wave & 3, ks = wave >> 2;
  auto &parts = lds.stage[ks].parts;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;   // (same columns of I -> same XCD, as spmm_mfma)
  // (what the prologue reads of the kernel arguments, at once: see grid_args)
  asm volatile("" ::"s"(p.by_mt.mul), "s"(p.by_mt.shift), "s"(p.by_gz.mul), "s"(p.by_gz.shift),
               "s"(p.by_c2.mul), "s"(p.by_c2.shift),
               "s"(p.ntiles), "s"(p.a1), "s"(p.a3), "s"(p.adj0), "s"(p.rowoff), "s"(p.d1), "s"(p.c2), "s"(p.Wp), "s"(p.I), "s"(p.ldI), "s"(p.N));
  const int gz = p.a3 >> 5, mt = p.a1 * gz;
  const int stripe = rbgp_fast::quotient(slot, p.by_mt), in_tile = slot - stripe * mt;
  const int nt = xcd + 8 * stripe;
  if (nt >= p.ntiles) return;                   // (the whole workgroup)
  const int u1 = rbgp_fast::quotient(in_tile, p.by_gz), ub = (in_tile - u1 * gz) * 32 + wid * 8;   // tile row, the wave's first G_i vertex
  const int64_t n0 = int64_t(nt) * CW;
  const int h = lane >> 5, j = lane & 31;
  const int adj_lo = lane < p.d1 ? p.adj0[u1 * p.d1 + lane] : 0;
  const int adj_hi = lane + 64 < p.d1 ? p.adj0[u1 * p.d1 + lane + 64] : 0;
  // the lane's kept weights of a stage: vertex ub + lane / 8, steps lane % 8 (+ 8), four rows each; where they go
  int to[IT], late[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = p.rowoff[(ub + (lane >> 3)) * KS + (lane & 7) + 8 * it];
    // in halfwords, row 0.  Sparse: step k or k + 16 is place k % 4 + 4 (k / 8) of operand half k / 4 % 2
    to[it] = SPARSE ? (((k >> 2) & 1) * 8 + (lane >> 3)) * 8 + (k & 3) + ((k >> 1) & 4)
                    : ((k >> 4) * 64 + ((k >> 3) & 1) * 8 + (lane >> 3)) * 8 + (k & 7);
    if constexpr (SPARSE) late[it] = k >> 4;
  }
  halfword *const wl = reinterpret_cast<halfword *>(wparts[wave]);
  // Row r of vertex v, operand half x lies at piece 16 r + ((8 x + v) ^ 4 r): the 16 pieces that an instruction writes (one r) and
  // the 16 that a quarter of a wave reads (four v, all r) are in different banks.
  auto row_to = [&](int base, int r) { return (base ^ 32 * r) + 128 * r; };
  const int own_w = 16 * (j & 3) + ((8 * h + (j >> 2)) ^ 4 * (j & 3));   // the lane's own piece
  auto no_weights = [&]() {
#pragma unroll
    for (int k = 0; k < 3 * WB; ++k) wparts[wave][k / WB][k % WB][lane] = u32x4{0, 0, 0, 0};
    __builtin_amdgcn_wave_barrier();
  };
  no_weights();
  int which = 0;                                // the sparse MFMA's index operand: 2-bit places in the groups of four
  if constexpr (SPARSE) {
#pragma unroll
    for (int it = 0; it < IT; ++it) wl[to[it]] = halfword(late[it]);
    __builtin_amdgcn_wave_barrier();
    const u32x4 at = wparts[wave][0][0][8 * h + (j >> 2)];   // (the four rows of a vertex have the same steps)
#pragma unroll
    for (int e = 0; e < 8; ++e) which |= (2 * (e & 1) + int((at[e / 2] >> (16 * (e & 1))) & 1u)) << (2 * e);
    __builtin_amdgcn_wave_barrier();
    no_weights();
  }
  const int nstages = p.d1 * p.c2;
  const float *const wbase = p.Wp + ((int64_t(u1) * nstages) * p.a3 + ub + (lane >> 3)) * 64 + (lane & 7) * 4;
  const int row_bytes = int(p.ldI * 4);         // (32 rows and a column tile stay below 2^31 bytes: checked by the host)
  const int own_t = wid % NT, own_u = NT == 2 ? wid >> 1 : 0;   // the column block, and first 16 steps, that the wave splits
  const int voff = (h * 8 + (SPARSE ? 4 : 16) * own_u) * row_bytes + (32 * own_t + j) * 4;
  auto first_row = [&](int s) {
    const int j1 = rbgp_fast::quotient(s, p.by_c2), v1 = j1 < 64 ? __builtin_amdgcn_readlane(adj_lo, j1) : __builtin_amdgcn_readlane(adj_hi, j1 - 64);
    return (int64_t(v1) * p.c2 + (s - j1 * p.c2)) * 32;
  };
  // sparse: row e of both halves of the stage in braw[2 e], braw[2 e + 1]; else row e of block own_u + u in braw[8 u + e]
  float braw[8 * TU];
  f32x4 araw[IT];
  // extent: to the last column of the stage's last row (columns past it read zeros or the next row; never stored)
  auto stage_rsrc = [&](int s) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.I + first_row(s) * p.ldI + n0), 0,
                                             31 * row_bytes + int((p.N - n0) * 4 < CW * 4 ? (p.N - n0) * 4 : CW * 4), kRsrcFlags);
  };
  auto load_round = [&](int s) {                // (the last round loads its own stage again)
    const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
#pragma unroll
    for (int it = 0; it < IT; ++it)
      araw[it] = *reinterpret_cast<const f32x4_u *>(wbase + int64_t(s) * p.a3 * 64 + 32 * it);
#pragma unroll
    for (int e = 0; e < 8 * TU; ++e)
      braw[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, voff, (SPARSE ? 16 * (e % 2) + e / 2 : 16 * (e / 8) + e % 8) * row_bytes, 0));
  };
  f32x16 acc[NT], cor[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = cor[t][i] = 0.f;
  load_round(ks < nstages ? ks : 0);
  for (int r = 0; r < nstages; r += KSP) {
    const int s = r + ks, buf = (r / KSP) & 1;
    const bool mine = KSP == 1 || s < nstages;
#pragma unroll
    for (int u = 0; u < TU; ++u) {              // (sparse: groups of four: the rows of steps k, k + 16, k + 1, k + 17)
      const float x[8] = {braw[8 * u], braw[8 * u + 1], braw[8 * u + 2], braw[8 * u + 3],
                          braw[8 * u + 4], braw[8 * u + 5], braw[8 * u + 6], braw[8 * u + 7]};
      const Split b = split8(x);
#pragma unroll
      for (int k = 0; k < 3; ++k) parts[buf][own_u + u][own_t][k][lane] = __builtin_bit_cast(u32x4, b.p[k]);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        uint32_t part[3];
        split2(araw[it][r], araw[it][r + 1], part);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          wl[k * 512 * WB + row_to(to[it], r)] = halfword(part[k]);
          wl[k * 512 * WB + row_to(to[it], r + 1)] = halfword(part[k] >> 16);
        }
      }
    load_round(s + KSP < nstages ? s + KSP : mine ? s : 0);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
    if (!mine) break;                           // (the last round)
    if constexpr (SPARSE) {
      bf16x8 a[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) a[k] = __builtin_bit_cast(bf16x8, wparts[wave][k][0][own_w]);
#pragma unroll
      for (int t = 0; t < NT; t += 2) {
        bf16x16 b[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 3; ++k) b[x][k] = joined(parts[buf][0][t + x][k][lane], parts[buf][1][t + x][k][lane]);
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            f32x16 &d = k == 0 ? acc[t + x] : cor[t + x];
            d = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a[pa[k]], b[x][pb[k]], d, which, 0, 0);
          }
      }
    }
#pragma unroll
    for (int u = 0; u < (SPARSE ? 0 : 2); ++u) {
      bf16x8 a[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) a[k] = __builtin_bit_cast(bf16x8, wparts[wave][k][u % WB][own_w]);
#pragma unroll
      for (int t = 0; t < NT; t += 2) {
        bf16x8 b[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 3; ++k) b[x][k] = __builtin_bit_cast(bf16x8, parts[buf][u][t + x][k][lane]);
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            f32x16 &d = k == 0 ? acc[t + x] : cor[t + x];
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[k]], b[x][pb[k]], d, 0, 0, 0);
          }
      }
    }
    __builtin_amdgcn_wave_barrier();            // (the next stage's weights come after these reads: one wave, in order)
  }
  // register i of block t: row 8 (i / 4) + 4 h + i % 4 of the wave's 32 (vertex ub + row / 4, row % 4), column 32 t + j
  int64_t row_of[4];                            // row of O of row r of G_i vertex 0 (four rows a vertex: a4 is 1, 2 or 4)
  const int lga4 = p.a4 >> 1;
#pragma unroll
  for (int r = 0; r < 4; ++r) row_of[r] = (int64_t(u1) * p.a2 + (r >> lga4)) * p.a3 * p.a4 + (r & (p.a4 - 1));
  uint32_t again[TU] = {};                      // sums that are not finite: bit 16 (t % 2) + i of word t / 2
#pragma unroll
  for (int t = 0; t < NT; ++t) add_up(acc[t], cor[t]);
  if constexpr (KSP > 1) {
    __syncthreads();
    if (ks)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) lds.red[ks - 1][t][i][wid][lane] = acc[t][i];
    __syncthreads();
    if (ks) return;                             // (no barrier from here on)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int k = 0; k < KSP - 1; ++k) acc[t][i] += lds.red[k][t][i][wid][lane];
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bool in = n0 + 32 * t + j < p.N;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t m = row_of[i % 4] + (ub + 2 * (i / 4) + h) * p.a4;
      const bool finite = acc[t][i] * 0.f == 0.f;
      if (in && finite) __builtin_nontemporal_store(acc[t][i], p.O + m * p.ldO + n0 + 32 * t + j);
      if (in && !finite) again[t / 2] |= 1u << (16 * (t % 2) + i);
    }
  }
  uint32_t any = 0;
#pragma unroll
  for (int x = 0; x < TU; ++x) any |= again[x];
  if (!__builtin_amdgcn_ballot_w64(any != 0)) return;   // (no barrier from here on)
  // The sums left out, from the kept weights alone and in the order of spmm_mfma: a G_i vertex of the wave after the other,
  // four rows x 64 columns per MFMA, the lane on the columns lane (and 64 + lane).
  for (int v = 0; v < 8; ++v) {
    uint32_t need[TU], some = 0;                // rows of the vertex that miss the lane's columns
#pragma unroll
    for (int x = 0; x < TU; ++x) {
      need[x] = (uint32_t(__builtin_amdgcn_ds_bpermute(((v & 1) * 32 + j) * 4, int(again[x]))) >> (16 * h + 4 * (v >> 1))) & 15u;
      some |= need[x];
    }
    if (!__builtin_amdgcn_ballot_w64(some != 0)) continue;
    const int ui = ub + v;
    const int ro = p.rowoff[ui * KS + lane % KS] * row_bytes;
    const float *const wv = p.Wp + ((int64_t(u1) * nstages) * p.a3 + ui) * 64 + lane;
    float wnext, bnext[TU][KS];
    auto load_stage = [&](int s) {
      const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
      wnext = wv[int64_t(s) * p.a3 * 64];
#pragma unroll
      for (int b = 0; b < KS; ++b)
#pragma unroll
        for (int x = 0; x < TU; ++x)
          bnext[x][b] = __uint_as_float(
              __builtin_amdgcn_raw_buffer_load_b32(rb, __builtin_amdgcn_readlane(ro, b) + (64 * x + lane) * 4, 0, 0));
    };
    f32x4 sum[TU];
#pragma unroll
    for (int x = 0; x < TU; ++x) sum[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    load_stage(0);
    for (int s = 0; s < nstages; ++s) {
      const float w = wnext;
      float b[TU][KS];
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int x = 0; x < TU; ++x) b[x][k] = bnext[x][k];
      load_stage(s + 1 < nstages ? s + 1 : s);
      static_for<0, KS>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int x = 0; x < TU; ++x) sum[x] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, b[x][k], sum[x], 4, k, 0);
      });
    }
#pragma unroll
    for (int x = 0; x < TU; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = row_of[r] + int64_t(ui) * p.a4;
        if (need[x] >> r & 1u) p.O[m * p.ldO + n0 + 64 * x + lane] = sum[x][r];
      }
  }
}

}  // namespace

rbgp_reg_fn rbgp_reg_split_kernel(int RW, bool sparse) {
  return RW == 4 ? (sparse ? spmm_reg_split_shared<true> : spmm_reg_split_shared<false>) : RW == 1 ? spmm_reg_split : nullptr;
}

namespace {

template <int NT, int KSP>
rbgp_split_tile_fn pick_split_tile(int KS, bool sparse) {
  return KS == 8    ? (sparse ? spmm_mfma_split<8, true, NT, KSP> : spmm_mfma_split<8, false, NT, KSP>)
         : KS == 16 ? (sparse ? spmm_mfma_split<16, true, NT, KSP> : spmm_mfma_split<16, false, NT, KSP>)
                    : nullptr;
}

}  // namespace

rbgp_split_tile_fn rbgp_mfma_split_kernel(int KS, bool sparse, int NT, int KSP) {
  return NT == 4 ? pick_split_tile<4, 1>(KS, sparse) : KSP == 1 ? pick_split_tile<2, 1>(KS, sparse) : pick_split_tile<2, 2>(KS, sparse);
}
