// Shared by the register-streaming MFMA kernels (fp32 and bf16 translation units):
// kernel parameter block and small device helpers.
#ifndef RBGP_REG_COMMON_H
#define RBGP_REG_COMMON_H

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "rbgp_fastdiv.h"

namespace rbgp_reg {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// fp32 -> bfloat16 bits, round to nearest, ties to even: the conversion instruction of gfx950
// (v_cvt_pk_bf16_f32, two values each), which the compiler selects for these casts.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ uint32_t bf16_bits(float x) { return bf16_pair(x, 0.f) & 0xffffu; }

struct RegParams {
  const float *Wp;         // packed weights (fp32, or bf16 bits for the bf16 kernels)
  const float *I;          // activations (same)
  float *O;                // fp32, or bf16 bits when obf16 is set (ldO counts elements of that type)
  int obf16;               // bf16 kernels: round the sums to bf16 when storing O
  int through;             // spmm_reg, whole lists: store rows of O through the caches
  const int32_t *rowtab;   // [a_i][NO*4]: stage-relative I row of each contraction step (padding -> 0); row_offset's table after it
  const int32_t *stages;   // [ncl][1+MG][tstride]: per stage the base row of the stage, then per
                           //   cluster member j_o * NSTG + (stage within the tile), the position of its
                           //   weight fragment among the member's fragments; -1 past the end (sentinel
                           //   stages) and when the member does not have the tile.  Wave k of the S that split a
                           //   list holds stage k + l * S in lane l.
  int tstride;             // 64, or 256 where a list has more than 60 stages (its last entry is always a sentinel)
  const int32_t *counts;   // [ncl] stages of each cluster (<= 60 per wave: <= 60 * S)
  const int32_t *members;  // [ncl][MG] tile rows of each cluster (-1: none)
  int64_t N, ldI, ldO;
  uint32_t w_bytes;        // extent of the packed weights (buffer descriptor)
  uint32_t row_bytes;      // ldI in bytes
  uint32_t n_bytes;        // N in bytes (N rounded up to a lane's load for bf16): extent of the last row of I
  int last_row, src_rows;  // K - 1; rows of I one stage spans
  // Fused 3x3 convolution (fp32 kernels): I is not materialised; row k = 9 * channel + tap of it is
  // read from the zero-padded activations X[channel][image][H+2][W+2].  Then the "row" unit of the
  // three fields above is a channel (row_bytes = bytes of one channel of X, last_row = channels - 1,
  // src_rows = channels one stage spans, n_bytes = row_bytes) and rowtab holds byte offsets
  // (channel and tap shift) instead of rows.
  int conv;                // 1: fused convolution
  int conv_h, conv_w;      // image height and width (W a multiple of 4)
  const int32_t *colbase;  // fused convolution: byte offset, inside a channel of X, of the first pixel of every
                           //   group of columns one lane loads (4, or 8 with the wide bf16 tile); padded to whole tiles
  int a2, a3, a4, R;
  int fpm;                 // weight fragments per member: d_o * NSTG
  int no4, kcr, frag_bytes, nq;   // entries of a G_i vertex's row table (all register kernels: row_offset); split-operand and shared
                           //   bf16 kernels: how many are steps, bytes of one weight fragment, blocks of 16 (bf16: 32) steps of a stage
  const int32_t *pairs;    // split operands, filled masks whose kept weights share the steps of a stage two by two: [fold][2][16],
                           //   see rbgp_reg_pairs
  int fold;                // tile rows per row of G_o
  int rowofs[16];          // output row of weight row r of a group, relative to its (tile row, u_i) base (masks without merged rows)
  int tm;                  // rows of one tile row: a_r * a_i * a_b
  int ntiles;              // column tiles: ceil(N / columns per wave)
  int lgS;                 // log2 of the waves that share a column tile (split of the stage list)
  int ncl;                 // clusters of tile rows (pairing kernel: quads)
  // (spmm_reg_rows: ncl = rows of G_o, ct_cnt = longest stage list)
  int ct, ct_cnt;          // fp32 kernels with stages of up to 8 steps: column tiles a wave takes one after the other (1 elsewhere)
                           //   and, when that is more than one, the stages of every cluster's list (all equal, a multiple of 4)
  // Workgroups (one-dimensional grid) are dealt round-robin to the 8 XCDs, so workgroup id & 7 is the XCD, each with
  // its own L2; within an XCD they start in the order of their ids.  A unit is a (G_i vertex, group of column
  // tiles) pair; the clusters of a unit are always neighbours on one XCD (they read the same rows of I).  order:
  //  2  column group g on XCD g & 7, all G_i vertices of a column group together: the workgroups that run at the same
  //     time read neighbouring columns on all eight XCDs (long runs of every row of I are wanted at once, which the
  //     memory likes), and G_i vertices that share rows of I share an L2.  For batches of at least 8 column groups.
  //  1  the units in (G_i vertex, column group) order, dealt to the XCDs in blocks of per_xcd items: an XCD reads one
  //     wide contiguous span of the rows of its G_i vertices.  Where every row of I belongs to one G_i vertex (right
  //     degree 1) and the batch is a few dozen column groups: on the VGG19 conv5 shape the XCDs then finish
  //     together, with order 2 every other XCD ran 1.4 us longer.
  //  0  as 1 in (column group, G_i vertex) order: small batches whose G_i vertices share rows of I.
  int per_xcd;             // items (cluster, unit) per XCD
  int ngroups;             // groups of column tiles (one group per workgroup)
  int order;
  int inner;               // G_i vertices, order 1: groups of column tiles
  rbgp_fast::Div by_ncl, by_inner;   // (set_grid)
  rbgp_fast::Div by_ct_cnt;
  rbgp_fast::Div by_row, by_r, by_a4;   // spmm_reg_rows: a3 R, R, a4
};

// The fields that wg_coord divides by; after ncl, a3, ngroups and order.
inline void set_grid(RegParams *p) {
  p->inner = p->order == 1 ? p->ngroups : p->a3;
  p->by_ncl = rbgp_fast::div_by(p->ncl);
  p->by_inner = rbgp_fast::div_by(p->inner);
}

constexpr int kRsrcFlags = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)
constexpr int kOob = 0x40000000;        // byte offset beyond any packed weight buffer (reads return 0)

// What a prologue reads of the kernel arguments, requested at once: left to where they are used, they arrive in three or four scalar
// loads that wait for one another.  Before wg_coord.
__device__ __forceinline__ void grid_args(const RegParams &p) {
  asm volatile("" ::"s"(p.order), "s"(p.per_xcd), "s"(p.ncl), "s"(p.inner), "s"(p.by_ncl.mul), "s"(p.by_ncl.shift), "s"(p.by_inner.mul),
               "s"(p.by_inner.shift), "s"(p.ngroups), "s"(p.a3), "s"(p.ntiles));
}
__device__ __forceinline__ void table_args(const RegParams &p) {
  asm volatile("" ::"s"(p.order), "s"(p.per_xcd), "s"(p.ncl), "s"(p.inner), "s"(p.by_ncl.mul), "s"(p.by_ncl.shift), "s"(p.by_inner.mul),
               "s"(p.by_inner.shift), "s"(p.ngroups), "s"(p.a3), "s"(p.ntiles), "s"(p.lgS), "s"(p.rowtab), "s"(p.stages), "s"(p.counts),
               "s"(p.members), "s"(p.tstride), "s"(p.no4), "s"(p.conv), "s"(p.Wp), "s"(p.I), "s"(p.w_bytes), "s"(p.row_bytes),
               "s"(p.n_bytes), "s"(p.last_row), "s"(p.src_rows), "s"(p.fpm), "s"(int(p.ldI)));
}

// (cluster, G_i vertex, group of column tiles) of this workgroup; false: none (the workgroup leaves)
struct WgCoord {
  int cl, u3, ntq;
};
__device__ __forceinline__ bool wg_coord(const RegParams &p, WgCoord *c) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int item = (p.order == 2 ? 0 : xcd * p.per_xcd) + slot;
  const int unit = rbgp_fast::quotient(item, p.by_ncl);
  c->cl = item - unit * p.ncl;
  const int hi = rbgp_fast::quotient(unit, p.by_inner), lo = unit - hi * p.inner;
  c->u3 = p.order == 1 ? hi : lo;
  c->ntq = p.order == 1 ? lo : p.order == 2 ? xcd + 8 * hi : hi;
  return p.order == 1 ? hi < p.a3 : c->ntq < p.ngroups;
}

// rowofs[r], or the same of G_i vertex u3 where it depends on that (rbgp_mask::merged).  Read from the row table for all masks: a
// choice between two tables in the prologue puts a latency of the scalar loads before the first vector loads (us against rowofs alone:
// conv5 fp32, 2048 columns, +0.46, conv3 bf16, 8192 columns, +0.18; from one table -0.07 and -0.11, one image of a VGG19 layer in bf16
// 6.78 -> 6.55).
__device__ __forceinline__ int row_offset(const RegParams &p, int u3, int r) {
  return p.rowtab[p.a3 * p.no4 + u3 * 16 + r];
}

// A lane's four neighbouring columns of a row of O in one store, whatever the alignment of the row (that of an element): rows of an odd
// number of columns begin anywhere, and column by column their stores were a quarter of some kernels (4096 x 4096 at 1/8 in bf16, 4001
// columns 37.5 us -> 31, 3374 54 -> 47; at 1/4, 331 columns 23.1 -> 20.9; fp32, 3331 columns 213 -> 202).  PAST: past the caches.
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef unsigned int u32x2_out __attribute__((ext_vector_type(2)));
typedef u32x2_out u32x2_any __attribute__((aligned(2)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));
template <bool PAST = true>
__device__ __forceinline__ void store_x4(float *o, const f32x4 &v) {
  if constexpr (PAST) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any *>(o));
  else *reinterpret_cast<f32x4_any *>(o) = v;
}
template <bool PAST = true>
__device__ __forceinline__ void store_x4(uint16_t *o, const f32x4 &v) {
  const u32x2_out w = {bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3])};
  if constexpr (PAST) __builtin_nontemporal_store(w, reinterpret_cast<u32x2_any *>(o));
  else *reinterpret_cast<u32x2_any *>(o) = w;
}

// Element offsets of the weight rows that a lane of half h holds of a 16-row group in the 32x32 MFMAs' layout, 8 (x / 4) + 4 h + x % 4,
// from the group's first row of O; -1: no such row.  rov: row_offset of row lane % 16.
__device__ __forceinline__ void row_offsets(int64_t (&at)[8], int rov, int h, int rows, int64_t ldO) {
  int ro[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) ro[x] = __builtin_amdgcn_ds_bpermute((8 * (x / 4) + 4 * h + x % 4) * 4, rov);
#pragma unroll
  for (int x = 0; x < 8; ++x) at[x] = 8 * (x / 4) + 4 * h + x % 4 < rows ? ro[x] * ldO : -1;
}

__device__ __forceinline__ f32x4 load_x4(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
  return f32x4{__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3])};
}

}  // namespace rbgp_reg

namespace rbgp_reg {
// Parameter block of the lo/hi pairing kernel (rbgp_mfma_reg_dual.hip): RegParams plus one table
// buffer in device memory laid out for few, wide loads (a wave reads it with 7 load instructions; 2048
// waves reading the same few KB with 25 narrow loads each is a burst of 50 000 load instructions at the
// head of every launch).  Measured alternatives for the 1.4 us between wave start and "tables there":
// tables inside the kernel arguments read by vector loads 1.6 us, by scalar loads 2.7 - 5 us (only the
// first bytes of the arguments arrive fast, 0.3 us); 16 copies of the buffer on different L2 channels
// 1.6 - 2.3 us (the one copy is fetched from memory once and then shared; it is not a hot spot).
struct DualParams {
  RegParams r;          // (rowtab / stages / counts / members are not used)
  const int32_t *tab;   // first, for every G_i vertex: [4 lane groups][rt_stride], the stage-relative row of I of step 4 * o + g at
                        //   [g][o], and 16 entries as row_offset gives them
  int rt_stride;        // NO rounded up to 4
  int cmax;             // stages stored per wave (>= the longest stage list)
  int o_stages;         // word offsets into tab of: stages [quad][x][y][cmax][4] (base row of I, position of L_x's
                        //   weight fragment, of H_y's, unused)
  int o_quads;          //   [quad][8]: L0, L1, H0, H1 (-1: none), then the stage counts of waves (0,0) (0,1) (1,0) (1,1)
};
}  // namespace rbgp_reg

namespace rbgp_reg {
// Parameter block of spmm_mfma_split (rbgp_mfma_reg_split.hip): the LDS family's weights and tables, four rows per column
// set (RB = 1), 32 rows of I per stage.
struct SplitTileParams {
  const float *Wp, *I;
  float *O;
  const int32_t *adj0;     // [a_o][d_o], d_o <= 128
  const int32_t *rowoff;   // [a_i][KS]: row of the stage of each step
  int64_t N, ldI, ldO;
  int a1, a2, a3, a4, d1, c2;
  int ntiles;              // column tiles of 32 NT
  rbgp_fast::Div by_mt, by_gz, by_c2;   // workgroups of a column tile, of a tile row (a3 / 32)
};
}  // namespace rbgp_reg

namespace rbgp_reg {
// Parameter block of conv_tile (rbgp_conv_tile.hip).
struct ConvTileParams {
  const void *Wp, *X;
  void *O;
  const uint64_t *tiles;   // [3][rows] tile columns of a row of G_o (at most 64 of them), a bit each: all; every other one, from the first
                           //   and from the second on.  rows: a_o rounded up to a multiple of four, the last ones empty
  int rows;
  const int4 *sel;         // [a_i] byte selectors and index operand of a G_i vertex (see the kernel)
  int64_t ldO, chan;       // elements of one channel of X
  uint32_t w_bytes;
  int n, ntiles;           // pixels, column tiles
  int h, w, w2, hw;        // image height, width, width + 2, height * width
  int a1, a2, a3, a4, d1, R, RS, frag_bytes;
  int chunk;               // tiles staged at once
  int obf16;
  rbgp_fast::Div by_per, by_hw, by_w, by_R, by_a4;   // per: workgroups of one column tile
};
}  // namespace rbgp_reg

typedef void (*rbgp_reg_fn)(rbgp_reg::RegParams);
typedef void (*rbgp_conv_tile_fn)(rbgp_reg::ConvTileParams);
// bf16 fused convolution with the channels of a tile as an image in LDS (rbgp_conv_tile.hip), 32 T pixels (T = 1, 2) and 4 S waves
// (S = 1, 2) per workgroup
rbgp_conv_tile_fn rbgp_conv_tile_kernel(int T, int S);
typedef void (*rbgp_split_tile_fn)(rbgp_reg::SplitTileParams);
typedef void (*rbgp_dual_fn)(rbgp_reg::DualParams);
// bf16 kernel for KC contraction steps per stage, RS weight rows per tile row, G 16-row
// groups per wave and CW (64 or 128) columns per wave; nullptr when that combination is not built.
rbgp_reg_fn rbgp_reg_bf16_kernel(int KC, int RS, int G, int CW);
// the same with one register set (two waves per SIMD); nullptr where that variant is not built
rbgp_reg_fn rbgp_reg_bf16_lean_kernel(int KC, int RS, int G, int CW);
// a wave's list in two chains of sums: 64 columns with two register sets, 128 with one
rbgp_reg_fn rbgp_reg_bf16_half_kernel(int KC, int RS, int CW);
// bf16 kernel of workgroups of RV x (4 / RV) waves, each 2 PR tile rows x 128 columns, that pass I through LDS;
// nullptr: not built
rbgp_reg_fn rbgp_reg_bf16_shared_kernel(int RV, int PR);
// fp32 kernel on the bf16 matrix core (operands split in three), 128 columns per wave; RW = 1: a
// wave by itself, 4: the four waves of a workgroup share the columns (sparse: on the sparse MFMA, RegParams::pairs);
// nullptr: not built
rbgp_reg_fn rbgp_reg_split_kernel(int RW, bool sparse);
// fp32 kernel of workgroups that take all rows of a row of G_o (rbgp_mfma_reg_rows.hip) x 32 T columns: 2, or 3 for lists of up to
// four stages; nullptr: not built
rbgp_reg_fn rbgp_reg_rows_kernel(int T, bool far);
// kernel of workgroups of eight waves that share a stage list, on 16 columns (rbgp_mfma_reg_narrow.hip); nullptr: not built
rbgp_reg_fn rbgp_reg_narrow_kernel(int KC, int RS, bool bf16);
// LDS family, fp32, on the bf16 matrix core: KS kept steps of 32 per stage (8 or 16; sparse: never both k and k + 16), workgroups of
// 32 NT columns (2, 4) and 4 KSP waves (1, or 2 with NT = 2); nullptr: not built
rbgp_split_tile_fn rbgp_mfma_split_kernel(int KS, bool sparse, int NT, int KSP);
// fp32 kernel with lo/hi pairing of the tile rows (8-row halves; tables of rbgp_reg_dual in the
// stages / counts / members fields); nullptr when KC is not built.
rbgp_dual_fn rbgp_reg_dual_kernel(int KC);
// the same with a wave's list in two chains of sums (stages of 36 and 72 steps)
rbgp_dual_fn rbgp_reg_dual_half_kernel(int KC);

#endif
