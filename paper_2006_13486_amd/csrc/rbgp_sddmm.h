// Parameters of the weight-gradient kernels (rbgp_sddmm.hip, rbgp_sddmm_lines.hip).
#ifndef RBGP_SDDMM_H
#define RBGP_SDDMM_H

#include <cstdint>

#include "rbgp_fastdiv.h"

namespace rbgp_sddmm_detail {

struct SddmmParams {
  const void *dO, *I;
  float *out;               // [workgroups per unit][nnz] partial sums (dW itself when there is one)
  const int32_t *colrows;   // [c_o][EO]: tile rows that have tile column v_o, ascending
  const int32_t *colpos;    // [c_o][EO]: position of v_o in that tile row's adjacency list
  const int32_t *rowtab;    // [a_i][16 * NB]: stage-relative row of I of contraction step kk (padding -> 0)
  int64_t N, ld_dO, ldI, nnz;
  int64_t chunk;            // columns per range (a multiple of the columns per iteration)
  int EO, RBG;              // tile rows per tile column; groups of RB row groups per unit
  int nbt, halves;          // 16-step groups of a stage; workgroups that share them (each takes NB consecutive ones)
  int c1, order;            // sddmm_lines: columns of G_o; which units are neighbours (1: those of a G_i vertex, 0: of a tile column)
  int NSTG, stage_rows;     // stages per tile; rows of I between the bases of consecutive stages (VC * c_i * c_b)
  int tile_rows;            // rows of I per tile column (c_r * c_i * c_b)
  int a2, a3, a4, R, lgRS, MG, KCR, rowdeg;
  // "All of G_i" units (GI kernels): a unit is a (tile column, stage) and takes the rows of every G_i vertex
  // together -- 16-row groups run over (tile row of the list, u_i, row of R) -- against ALL rows of I the
  // stage spans, whether G_i connects them or not; the epilogue stores the kept products only.  For
  // masks with few rows per (tile column, u_i) (sparse G_o, small G_r, G_b) this fills the 16 MFMA rows
  // that would be padding, and every row of I is loaded once instead of once per adjacent u_i.
  int src_rows;             // gi: rows of I one stage spans (VC * c_i * c_b)
  const int32_t *spos;      // gi: [a_i][16 * NB]: position inside the stage's kept values of (u_i, stage row), -1: not kept
  // Fused 3x3 convolution (CONV kernels): I is not materialised; row k = 9 * channel + tap of it is read
  // from the zero-padded activations X[channel][image][H + 2][W + 2] (pointer I).
  const int32_t *colbase;   // element offset, inside a channel of X, of the first pixel of every group of
                            //   columns one lane loads (4 fp32 / 8 bf16), padded with valid offsets
  int64_t chan_elems;       // elements of one channel of X
  int64_t x_bytes;          // size of X
  int conv_w2;              // W + 2
  // workgroups that share the rows of I of a (tile column, stage) in sddmm_reg; the rest by name
  rbgp_fast::Div by_sharing, by_halves, by_RBG, by_a3, by_NSTG, by_c1, by_R, by_a4;
};

constexpr int kLinesWaves = 8;   // waves of a workgroup of sddmm_lines

}  // namespace rbgp_sddmm_detail

typedef void (*rbgp_sddmm_fn)(rbgp_sddmm_detail::SddmmParams);
// sddmm_lines with RB (1, 2) groups of 16 rows of dO and NB (1 to 3; bf16 also 4 and 5, with conv 6) groups of 16 steps per wave;
// far (conv): dO of 4 GiB and more; nullptr: not built
rbgp_sddmm_fn rbgp_sddmm_lines_kernel(int RB, int NB, bool bf16, bool conv, bool gi, bool far);

#endif
