// bf16 kernel of the register-streaming family for masks whose tile rows come in groups of 2, 4 or 8 with one stage
// list (rows of G_r moved into the tile-row index: filled masks, merged columns, transposed layers).
//
// spmm_reg_bf16 transposes the rows of I in registers for each of its waves (four v_perm_b32 per column and eight steps),
// loads I once per wave and multiplies 16 rows per MFMA.  Here the waves of a workgroup load and transpose every
// block of 32 contraction steps x 128 columns once between them and pass it through LDS in operand layout (16 bytes per
// lane, no bank conflicts); v_mfma_f32_32x32x16_bf16 multiplies twice as many rows per operand byte.  Same packed weights
// (an A operand is one 16-byte load, requested a round ahead), same stage lists, same order of the sums (results equal
// spmm_reg_bf16's bit for bit where that does not split its lists); one barrier per round, double-buffered.
//
// What bounds it: the traffic past the L2s (every XCD reads all packed weights of its columns; 5 TB/s with the stores,
// what a copy reaches) and LDS reads, which a wave of two row pairs (PR = 2) halves per product.  Measured, 4096^3, density
// 1/8, four rows per column set, fp32 output: 85 us -> 45 (740 TFLOP/s on the filled mask), bf16 output 72 -> 44; one wave
// group of 4 x 1 with PR = 1 56; three waves per SIMD with one buffer 57; two rounds of loads in flight 49 (against 50).  The
// stores' offsets ahead of the stores and descriptors that the compiler knows to be uniform: fp32 output 41.8 us -> 40.2, transposed
// VGG19 layer 3 at 1/2, 71 images 20 -> 17.5; rows of O in one store a lane whatever their alignment: store_x4.
#include <hip/hip_runtime.h>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"

using namespace rbgp_reg;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// RV x (4 / RV) waves along rows and columns of the output, each 2 PR tile rows x 128 columns; a round is RV blocks of 32
// steps, of which every wave loads one on one of the column tiles.
template <int RV, int PR>
__global__ __launch_bounds__(256, 2) void spmm_reg_bf16_shared(RegParams p) {
  constexpr int NTC = 4 / RV, CW = 128 * NTC;   // column tiles and columns of a workgroup
  constexpr int NB = RV;                        // blocks of a round: every wave stages one on one of the tiles
  constexpr int QB = 4 * 16 * 16;               // bytes of 32 steps of a packed fragment (16 rows)
  __shared__ __attribute__((aligned(16))) u32x4 parts[2][NB][NTC][2][4][64];   // [..][16 steps][column block][lane]
  __shared__ __attribute__((aligned(16))) int rowoff[3 * 32];                 // byte offset of a step's row of I
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int wr = wid / NTC, wc = wid % NTC;     // row group and column tile; as a loader, block and column tile
  table_args(p);
  WgCoord wg;
  if (!wg_coord(p, &wg)) return;                // (the whole workgroup)
  const int u1 = (wg.cl * RV + wr) * 2 * PR, u3 = wg.u3;   // first of the wave's 2 PR tile rows
  const int nt = wg.ntq;
  const int64_t n0 = int64_t(nt) * CW + wc * 128;   // the wave's first column
  const bool valid = n0 < p.N;
  const uint32_t n0b = p.conv ? 0u : uint32_t(n0 * 2);
  const int nq = p.nq;
  if (int(threadIdx.x) < nq * 32) {
    const int kk = threadIdx.x;
    const int r = kk < p.kcr ? p.rowtab[u3 * p.no4 + kk] : 0;
    // (< 2^31: checked by the host; padding steps lie past every extent and read zeros without a memory access)
    rowoff[kk] = kk >= p.kcr ? int(0x80000000u) : p.conv ? r : r * (int(p.ldI) * 2);
  }
  // one stage per lane (at most 64: checked by the host); both tile rows have the same list and the same positions
  const int TS = p.tstride;
  const int32_t *stg = p.stages + int64_t(u1) * 2 * TS + lane;
  const int tb = stg[0], tf = stg[TS];
  const int cnt = __builtin_amdgcn_readfirstlane(p.counts[u1]);
  const int rov = p.rowofs[lane & 15];
  const int o = lane >> 4, cg = lane & 15;      // as a loader: eight steps 8 o .. of a block, columns 8 cg ..
  const int h = lane >> 5, j = lane & 31;       // as an operand: eight steps 8 h .. of 16, row / column j
  const int col = p.conv ? p.colbase[valid ? int(n0 >> 3) + cg : 0] : cg * 16;
  const int fstr = p.fpm * p.a3 * p.frag_bytes;   // from one tile row's weights to the next one's
  const int alane = (j >> 4) * fstr + (h * 16 + (j & 15)) * 16;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void *>(static_cast<const void *>(p.Wp)), 0, p.w_bytes, kRsrcFlags);
  const int tbu = p.conv ? int(uint32_t(tb < 0 ? 0 : tb) / 9u) : (tb < 0 ? 0 : tb);
  const uint64_t i_first = reinterpret_cast<uint64_t>(p.I) + uint64_t(uint32_t(tbu)) * p.row_bytes + n0b;
  const int ib_lo = int(uint32_t(i_first)), ib_hi = int(uint32_t(i_first >> 32));
  // (to the last column of the stage's last row, so that an extent stays below 2^31: SRC rows of ldI do, checked by the host)
  const int rows_left = p.last_row - tbu < p.src_rows - 1 ? p.last_row - tbu : p.src_rows - 1;
  const int ib_ext = (tb >= 0 && valid) ? int(uint32_t(rows_left) * p.row_bytes + (p.n_bytes - n0b)) : 0;
  const int aoff = tf >= 0 ? ((u1 * p.fpm + tf) * p.a3 + u3) * p.frag_bytes : kOob;
  float *const out = p.O;
  const int64_t out_ld = p.ldO, out_n = p.N;
  const int out_tm = p.tm, out_a4 = p.a4, out_r = p.R, out_bf16 = p.obf16;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // block b of the list (stage s, its q-th 32 steps) in steps of one
  auto next = [&](int &s, int &q) {
    q = q + 1 < nq ? q + 1 : 0;
    s += q == 0;
  };
  u32x4 raw[8], A[NB][2][PR];
  auto load_i = [&](int s, int q) {             // (past the end: zero extent)
    const int tl = s < 63 ? s : 63;
    const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_lo, tl))) |
                          (uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_hi, tl))) << 32);
    const int ext = __builtin_amdgcn_readlane(ib_ext, tl);
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, s < cnt ? ext : 0, kRsrcFlags);
    const int4 *ro = reinterpret_cast<const int4 *>(rowoff + q * 32 + o * 8);
    const int4 r0 = ro[0], r1 = ro[1];
    const int off[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) raw[e] = __builtin_amdgcn_raw_buffer_load_b128(rb, off[e] + col, 0, 0);
  };
  auto load_a = [&](u32x4 (&a)[2][PR], int s, int q) {
    const int av = __builtin_amdgcn_readlane(aoff, s < 63 ? s : 63);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int y = 0; y < PR; ++y)
        a[u][y] = __builtin_amdgcn_raw_buffer_load_b128(rw, (s < cnt ? av : kOob) + alane + y * 2 * fstr + u * 512, q * QB, 0);
  };

  f32x16 acc[PR][4];
#pragma unroll
  for (int y = 0; y < PR; ++y)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[y][t][i] = 0.f;
  int si = 0, qi = 0, sa = 0, qa = 0;           // the next block this wave stages; the next block whose weights are requested
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    load_a(A[k], sa, qa);
    next(sa, qa);
    if (k < wr) next(si, qi);
  }
  // (uniform, which the compiler does not see of a count that starts at the wave's number: it put a loop over the lanes' descriptors
  // around every load of I, eight of 20 instructions each a round)
  if (RV > 1) si = __builtin_amdgcn_readfirstlane(si);
  if (RV > 1) qi = __builtin_amdgcn_readfirstlane(qi);
  load_i(si, qi);
  const int rounds = (cnt * nq + NB - 1) / NB;
  for (int r = 0; r < rounds; ++r) {
    const int buf = r & 1;
    constexpr unsigned LO = 0x05040100u, HI = 0x07060302u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {               // column 8 cg + i -> column block i % 4, lane (i / 4) * 16 + cg
      const int d = i / 2;
      const unsigned sel = i & 1 ? HI : LO;
      const u32x4 v = {__builtin_amdgcn_perm(raw[1][d], raw[0][d], sel), __builtin_amdgcn_perm(raw[3][d], raw[2][d], sel),
                       __builtin_amdgcn_perm(raw[5][d], raw[4][d], sel), __builtin_amdgcn_perm(raw[7][d], raw[6][d], sel)};
      parts[buf][wr][wc][o >> 1][i & 3][(o & 1) * 32 + (i >> 2) * 16 + cg] = v;
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) next(si, qi);
    load_i(si, qi);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    // groups of four operands, each read from LDS while the group before it is multiplied
    bf16x8 b[2][4];
    auto fetch = [&](auto gc) {
      constexpr int g = decltype(gc)::value;
#pragma unroll
      for (int t = 0; t < 4; ++t) b[g & 1][t] = __builtin_bit_cast(bf16x8, parts[buf][g / 2][wc][g % 2][t][lane]);
    };
    fetch(std::integral_constant<int, 0>{});
    static_for<0, 2 * NB>([&](auto gc) {
      constexpr int g = decltype(gc)::value, u = g % 2, k = g / 2;
      if constexpr (g + 1 < 2 * NB) fetch(std::integral_constant<int, g + 1>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int y = 0; y < PR; ++y)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[y][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, A[k][u][y]), b[g & 1][t], acc[y][t], 0, 0, 0);
      if constexpr (u == 1) {
        load_a(A[k], sa, qa);
        next(sa, qa);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // lane j holds the columns 8 (j % 16) + 4 (j / 16) .. + 3, register i the weight row 8 (i / 4) + 4 h + i % 4 of the 32: row
  // 8 (i / 4 % 2) + 4 h + i % 4 of the i / 8-th tile row.  Offsets first, then the stores, so that none of them waits for another.
  if (!valid) return;
  const bool aligned = out_ld % 4 == 0 && reinterpret_cast<uintptr_t>(out) % (out_bf16 ? 8 : 16) == 0;
  const int64_t n = n0 + 8 * (j & 15) + 4 * (j >> 4);
  const bool whole = n + 4 <= out_n;
  int64_t row_at[8];                            // of the eight rows of a tile row that the lane holds; -1: none
  row_offsets(row_at, rov, h, out_r, out_ld);
  const int64_t first = (int64_t(u1) * out_tm + u3 * out_a4) * out_ld + n, next_row = int64_t(out_tm) * out_ld;
  auto each = [&](auto put) {
#pragma unroll
    for (int y = 0; y < PR; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (row_at[i & 7] >= 0)
          put(first + (2 * y + (i >> 3)) * next_row + row_at[i & 7], f32x4{acc[y][0][i], acc[y][1][i], acc[y][2][i], acc[y][3][i]});
  };
  uint16_t *const out16 = reinterpret_cast<uint16_t *>(out);
  // (aligned rows past the caches; of others, the parts of a line that two workgroups write meet in the L2: 2047 columns 46.8 -> 44.9 us)
  if (whole && aligned && out_bf16)
    each([&](int64_t at, const f32x4 &v) { store_x4(out16 + at, v); });
  else if (whole && aligned)
    each([&](int64_t at, const f32x4 &v) { store_x4(out + at, v); });
  else if (whole && out_bf16)
    each([&](int64_t at, const f32x4 &v) { store_x4<false>(out16 + at, v); });
  else if (whole)
    each([&](int64_t at, const f32x4 &v) { store_x4<false>(out + at, v); });
  else {
    // (at most three columns left: one after the other for all rows, with one condition each; asked store by store, a tile that ends inside N
    // took 0.8 to 2.5 us longer: transposed VGG19 layer 6 at 1/2, 2368 columns 10.8 -> 9.3, O in bf16 10.7 -> 8.4, layer 3 at 1/2, 6143 11.6 -> 9.4)
#pragma unroll
    for (int w = 0; w < 3; ++w)
      if (n + w < out_n) {
        if (out_bf16) each([&](int64_t at, const f32x4 &v) { out16[at + w] = uint16_t(bf16_bits(v[w])); });
        else each([&](int64_t at, const f32x4 &v) { out[at + w] = v[w]; });
      }
  }
}

}  // namespace

rbgp_reg_fn rbgp_reg_bf16_shared_kernel(int RV, int PR) {
  if (PR == 2) return RV == 2 ? spmm_reg_bf16_shared<2, 2> : RV == 1 ? spmm_reg_bf16_shared<1, 2> : nullptr;
  return RV == 4 ? spmm_reg_bf16_shared<4, 1> : RV == 2 ? spmm_reg_bf16_shared<2, 1> : RV == 1 ? spmm_reg_bf16_shared<1, 1> : nullptr;
}
