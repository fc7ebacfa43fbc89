// fp32 product of the register-streaming family for masks with short stages and many rows per tile, on the sparse bf16
// matrix core with split operands (rbgp_split.h): the transposes of lowered 3x3 layers (dI = W_s^T x dO), whose tiles are
// nine times as high as they are wide.  A tile of G_o holds |G_r.U| |G_i.U| |G_b.U| rows (288 in VGG19's layers) and one
// stage of |G_r.V| |G_i.V| |G_b.V| = 4 x 4 x 2 rows of I, of which a row keeps two of every four (G_i: two edges, four
// columns).  spmm_reg walks such a tile once per G_i vertex, in stages of 16 steps, each row of I loaded |G_i.U| / 2 times
// for 9 to 12 of 16 MFMA rows: it waits for the load path.
//
// Here a workgroup takes all rows of a row of G_o (p.fold tile rows x G_i vertices x R) x 64 or 96 columns: every stage's 32 rows
// are loaded and split once, and stay in LDS (6 KB a stage for 32 columns); then every wave multiplies groups of 32 rows, whatever
// G_i vertices they belong to, with
// v_smfmac_f32_32x32x32_bf16: its index operand names the kept ones among the four columns of G_i, row by row, so that one
// instruction serves rows of different G_i vertices and no zero of G_i is multiplied.  The packed weights are those of
// spmm_reg, loaded four stages ahead.
// Operands: the lane of half h holds the kept weights of G_b vertex h, in groups of four (all G_i vertices of one G_r vertex
// v); the groups v = 0, 1 belong to rows of I in the lanes of half 0, v = 2, 3 to those of half 1.
//
// What bounds it: a workgroup's chain of latencies (tables, rows of I, four to eight stages of six dependent products each),
// and from a few hundred workgroups on the stores of O, 9 |G_r.U| rows for every 32 of I.  us, before -> after: VGG19 layer 6
// at density 1/4, 2368 columns 24.3 -> 16, 8192 49 -> 30; layer 9 at 1/4, 2048 columns 44 -> 27; layer 3, 32768 columns
// 62 -> 42; error against 64-bit sums 8.3e-8 -> 5.0e-8.  96 columns, where 64 leave some CUs two workgroups and others one: the
// products and stores of a block overlap the next one's in the other waves of the SIMD only, but a wave splits its weights once for
// three blocks and before it waits for the rows of I (layer 6, 2368 columns 16.2 -> 13.6).
// Tried: 32 and 128 columns a workgroup in the same manner (2368 columns, layer 6: 19 and 15.8), five and four waves of 96 columns
// (16.9, 22.3); waves of 32 columns at four waves per SIMD (15.7 / 32 / 29 / 48), two stages of weights ahead with 14 spilled
// registers (15.6 / 33 / 33 / 41), one edge of four (half of the weights zero; VGG19 conv5 24.9 -> 26.2), the next stage's
// operands prepared beside the products (21 / 39 / 32 / 53).
#include <hip/hip_runtime.h>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"
#include "rbgp_split.h"

using namespace rbgp_reg;
using namespace rbgp_split;

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2_s __attribute__((ext_vector_type(2)));
typedef f32x2_s f32x2_any __attribute__((aligned(4)));

constexpr int kAhead = 4;                       // stages of weights in flight
constexpr uint32_t kNone = 0xffffffffu;

// T = 2: 64 columns, a pair of them per lane, lists of up to twelve stages.  T = 3: 96 columns, a block of 32 at a time, lists of up
// to four stages.  FAR: a workgroup's rows of O lie 4 GiB apart and more: 64-bit offsets, made at the stores.
template <int T, bool FAR>
__global__ __launch_bounds__(576, 3) void spmm_reg_rows(RegParams p) {
  constexpr int CW = 32 * T;
  // [stage][column block][part][half of the 16 steps of a lane][lane], then what every row needs (info)
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), W = int(blockDim.x) >> 6;
  const int h = lane >> 5, j = lane & 31;
  int uo, nt;                                   // row of G_o, column tile (order 2: one on XCD tile % 8, as in wg_coord)
  if (p.order == 2) {
    const int slot = blockIdx.x >> 3;
    const int q = rbgp_fast::quotient(slot, p.by_ncl);
    nt = int(blockIdx.x & 7) + 8 * q;
    uo = slot - q * p.ncl;
  } else {
    nt = rbgp_fast::quotient(int(blockIdx.x), p.by_ncl);
    uo = int(blockIdx.x) - nt * p.ncl;
  }
  if (nt >= p.ntiles) return;                   // (the whole workgroup)
  const int64_t n0 = int64_t(nt) * CW;
  const int u1 = uo * p.fold, TS = p.tstride;
  // The tables in one go (lanes past the list hold sentinels), the rows of I as soon as those are there, then the weights: with a latency
  // after the other from the first to the last of these, and stores that waited for lookups, a wave took 22 100 cycles, now 18 900.
  const int32_t *stg = p.stages + int64_t(u1) * 2 * TS;
  const int tb0 = stg[lane], tf0 = stg[TS + lane], cnt0 = p.counts[u1];
  u32x4 *const parts = reinterpret_cast<u32x4 *>(lds);
  // of every row: its byte offset in O from the tile row's first row (FAR: in rows; kNone: no such row), then: its weights relative to a stage's,
  // the places of its G_i vertex's two edges (the index operand)
  uint32_t *const row_at = reinterpret_cast<uint32_t *>(lds + p.ct_cnt * (T * 6144));
  const int per_row = p.a3 * p.R, rows = p.fold * per_row, groups = (rows + 31) >> 5;
  int2 *const info = reinterpret_cast<int2 *>(row_at + groups * 32);
  const uint32_t ld_bytes = FAR ? 1u : uint32_t(p.ldO) * 4u;   // (a tile row of O is below 4 GiB unless FAR: checked by the host)
  // the edges of the G_i vertex of row x (of the rows that the thread prepares, the first)
  auto edges_of = [&](int x) {
    const int f = rbgp_fast::quotient(x, p.by_row), ui = rbgp_fast::quotient(x - f * per_row, p.by_r);
    const int32_t *rt = p.rowtab + (x < rows ? ui * p.no4 : 0);
    return int2{rt[0] >> 1, rt[2] >> 1};
  };
  int2 edges = edges_of(threadIdx.x);
  const int cnt = __builtin_amdgcn_readfirstlane(cnt0);
  const int tb = lane < cnt ? tb0 : 0, tf = lane < cnt ? tf0 : 0;   // (at most 12 stages)
  const int row_bytes = int(p.row_bytes);
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  auto stage_rsrc = [&](int s) {
    const uint32_t b = uint32_t(__builtin_amdgcn_readlane(tb, s));
    // (to the last column of the stage's last row; columns past it read zeros or the next row and are never stored)
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.I) + (uint64_t(b) * p.row_bytes >> 2) + n0, 0,
        int(31u * p.row_bytes + (p.n_bytes - uint32_t(n0) * 4u)), kRsrcFlags);
  };
  // row of the stage of step e of a lane of half hb: G_r vertex 2 hb + (e % 8) / 4, G_i vertex e % 4, G_b vertex e / 8
  auto row_of = [&](int hb, int e) { return ((2 * hb + (e % 8) / 4) * 4 + e % 4) * 2 + e / 8; };

  // two pieces of a row's fragment, steps of G_b vertex h: piece i is edge i of the row's G_i vertex, element v G_r vertex v
  struct A {
    f32x4 x[2];
  };
  auto a_of = [&](int r) {                      // its weights; kOob: no such row
    const int f = rbgp_fast::quotient(r, p.by_row), q = r - f * per_row, ui = rbgp_fast::quotient(q, p.by_r), i = q - ui * p.R;
    return r < rows ? ((u1 + f) * p.fpm * p.a3 + ui) * p.frag_bytes + i * 16 : kOob;
  };
  auto load_a = [&](A &a, int base, int s) {
    const int pos = __builtin_amdgcn_readlane(tf, s) * p.a3 * p.frag_bytes;
    a.x[0] = load_x4(rw, base + pos, 0);
    a.x[1] = load_x4(rw, base + pos, 512);
  };
  // The rows of I that the wave splits, of its first two items (more only where a workgroup has few waves): T = 2: a stage, a pair of
  // columns per lane; T = 3: a stage's column block.
  constexpr int NV = T == 3 ? 16 : 32;
  const int items = T == 3 ? cnt * T : cnt;
  auto load_rows = [&](float (&x)[NV], int item) {
    const int s = T == 3 ? item / 3 : item;
    const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if constexpr (T == 3) {
        x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, row_of(h, e) * row_bytes + (32 * (item - 3 * s) + j) * 4, 0, 0));
      } else {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rb, row_of(h, e) * row_bytes + j * 8, 0, 0);
        x[e] = __uint_as_float(v[0]);
        x[16 + e] = __uint_as_float(v[1]);
      }
    }
  };
  float x0[NV], x1[NV];
  if (wid < items) load_rows(x0, wid);
  if (wid + W < items) load_rows(x1, wid + W);
  A ring[kAhead];
  int a_base = a_of(wid * 32 + j) + h * 256;
#pragma unroll
  for (int d = 0; d < kAhead; ++d) load_a(ring[d], d < cnt ? a_base : kOob, d < cnt ? d : 0);

  for (int x = threadIdx.x; x < groups * 32; x += blockDim.x) {
    const int f = rbgp_fast::quotient(x, p.by_row), q = x - f * per_row, ui = rbgp_fast::quotient(q, p.by_r), i = q - ui * p.R;
    const int ia = rbgp_fast::quotient(i, p.by_a4);
    const bool in = x < rows;
    const int which = in ? (edges.x | edges.y << 2) * 0x1111 : 0;
    if (x + int(blockDim.x) < groups * 32) edges = edges_of(x + int(blockDim.x));
    row_at[x] = in ? uint32_t(f * p.tm + ui * p.a4 + ia * p.a3 * p.a4 + i - ia * p.a4) * ld_bytes : kNone;
    info[x] = int2{a_of(x), which};
  }
  auto keep = [&](const float (&x)[NV], int item) {
#pragma unroll
    for (int half = 0; half < NV / 8; ++half) {   // (T = 2: two column blocks)
      const int block = T == 3 ? item : item * 2 + half / 2;
      const float y[8] = {x[8 * half], x[8 * half + 1], x[8 * half + 2], x[8 * half + 3],
                          x[8 * half + 4], x[8 * half + 5], x[8 * half + 6], x[8 * half + 7]};
      const Split b = split8(y);
#pragma unroll
      for (int k = 0; k < 3; ++k) parts[((block * 3 + k) * 2 + half % 2) * 64 + lane] = __builtin_bit_cast(u32x4, b.p[k]);
    }
  };
  if (wid < items) keep(x0, wid);
  if (wid + W < items) keep(x1, wid + W);
  for (int item = wid + 2 * W; item < items; item += W) {
    load_rows(x0, item);
    keep(x0, item);
  }
  auto weights = [&](const A &a) {
    const float w[8] = {a.x[0][0], a.x[1][0], a.x[0][1], a.x[1][1], a.x[0][2], a.x[1][2], a.x[0][3], a.x[1][3]};
    return split8(w);
  };
  // sums of a column block (f32x16 pair) with one stage's weights
  auto multiply = [&](const Split &a, int block, int which, f32x16 &acc, f32x16 &cor) {
    constexpr int pa[6] = {0, 0, 1, 1, 0, 2}, pb[6] = {0, 1, 0, 1, 2, 0};
    bf16x16 b[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) b[k] = joined(parts[((block * 3 + k) * 2) * 64 + lane], parts[((block * 3 + k) * 2 + 1) * 64 + lane]);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      f32x16 &c = k == 0 ? acc : cor;
      c = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a.p[pa[k]], b[pb[k]], c, which, 0, 0);
    }
  };
  // the tile row's first row of O, at the workgroup's first column; register i of the accumulators is row 8 (i / 4) + 4 h + i % 4 of a
  // group
  unsigned char *const out = reinterpret_cast<unsigned char *>(p.O + int64_t(u1) * p.tm * p.ldO + n0);
  const int64_t out_n = p.N, far_ld = p.ldO * 4;
  // Past the caches only where rows begin at whole 64 bytes: of others, the parts of a line that two workgroups write meet in the L2
  // (us, past the caches / through them: layer 6 at 1/4, 8128 columns, rows of 8144 27.2 / 28.8, 8136 39.6 / 28.5, 8129 50.6 / 29.9;
  // layer 3, 16320, rows of 16336 25.3 / 23.2, 16321 47.2 / 26.4; 96 columns, 2304, rows of 2320 12.2 / 13.7, 2305 15.7 / 14.1)
  const bool past = p.ldO % 16 == 0 && reinterpret_cast<uintptr_t>(p.O) % 64 == 0;
  auto place = [&](uint32_t at, uint32_t column) {
    return reinterpret_cast<float *>(out + (FAR ? uint64_t(at) * uint64_t(far_ld) : uint64_t(at)) + column);
  };
  auto rows_at = [&](uint32_t (&at)[16], int g) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const u32x4 v = *reinterpret_cast<const u32x4 *>(row_at + g * 32 + 8 * x + 4 * h);
#pragma unroll
      for (int y = 0; y < 4; ++y) at[4 * x + y] = v[y];
    }
  };
  if constexpr (T == 3) {
    // (the first group's weights are split before the wave waits for the others)
    Split a[kAhead];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) a[d] = weights(ring[d]);
    __syncthreads();
    for (int g = wid; g < groups; g += W) {
      const int which = info[g * 32 + j].y;
      uint32_t at[16];
      rows_at(at, g);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        f32x16 acc, cor;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = cor[i] = 0.f;
#pragma unroll
        for (int d = 0; d < kAhead; ++d)
          if (d < cnt) multiply(a[d], d * T + t, which, acc, cor);
        const int64_t n = n0 + 32 * t + j;
        if (__builtin_amdgcn_ballot_w64(add_up(acc, cor) && n < out_n)) {   // (as below, with the one block)
          uint64_t left = __builtin_amdgcn_ballot_w64(row_at[g * 32 + j] != kNone);
          while (left) {
            const int pair = __builtin_amdgcn_readlane(which, __builtin_ctzll(left));
            left &= ~__builtin_amdgcn_ballot_w64(which == pair);
#pragma unroll
            for (int i = 0; i < 16; ++i) cor[i] = 0.f;
            for (int s = 0; s < cnt; ++s) {
              const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
              A aw;
              load_a(aw, a_base, s);
#pragma unroll
              for (int w = 0; w < 4; ++w)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(
                      rb, ((w * 4 + (pair >> (2 * e) & 3)) * 2 + h) * row_bytes + (32 * t + j) * 4, 0, 0);
                  cor = __builtin_amdgcn_mfma_f32_32x32x2f32(aw.x[e][w], __uint_as_float(x), cor, 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const bool mine = info[g * 32 + 8 * (i / 4) + 4 * h + i % 4].y == pair;
              acc[i] = acc[i] * 0.f == 0.f || !mine ? acc[i] : cor[i];
            }
          }
        }
        if (n < out_n && past) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (at[i] != kNone) __builtin_nontemporal_store(acc[i], place(at[i], uint32_t(128 * t + 4 * j)));
        } else if (n < out_n) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (at[i] != kNone) *place(at[i], uint32_t(128 * t + 4 * j)) = acc[i];
        }
      }
      if (g + W < groups) {
        a_base = info[(g + W) * 32 + j].x + h * 256;
#pragma unroll
        for (int d = 0; d < kAhead; ++d) load_a(ring[d], d < cnt ? a_base : kOob, d < cnt ? d : 0);
#pragma unroll
        for (int d = 0; d < kAhead; ++d) a[d] = weights(ring[d]);
      }
    }
    return;
  }
  __syncthreads();

  const bool whole = n0 + 2 * j + 2 <= out_n;
  for (int g = wid; g < groups; g += W) {
    const int which = info[g * 32 + j].y, base = a_base;
    a_base = g + W < groups ? info[(g + W) * 32 + j].x + h * 256 : kOob;
    f32x16 acc[2], cor[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = cor[t][i] = 0.f;
    for (int s0 = 0; s0 < cnt; s0 += kAhead) {
#pragma unroll
      for (int d = 0; d < kAhead; ++d) {
        const int s = s0 + d;
        if (s < cnt) {
          const Split a = weights(ring[d]);
          const bool more = s + kAhead < cnt;
          load_a(ring[d], more ? base : a_base, more ? s + kAhead : d);
#pragma unroll
          for (int t = 0; t < 2; ++t) multiply(a, s * 2 + t, which, acc[t], cor[t]);
        }
      }
    }
    bool again = false;
#pragma unroll
    for (int t = 0; t < 2; ++t) again |= add_up(acc[t], cor[t]) && n0 + 2 * j + t < out_n;
    if (__builtin_amdgcn_ballot_w64(again)) {   // (wave-uniform; no barrier inside)
      // The rows of one pair of edges at a time, with the rows of I at these edges only: a row of I that is not finite must not
      // meet a zero in the place of a weight.
      uint64_t left = __builtin_amdgcn_ballot_w64(row_at[g * 32 + j] != kNone);
      while (left) {
        const int pair = __builtin_amdgcn_readlane(which, __builtin_ctzll(left));
        left &= ~__builtin_amdgcn_ballot_w64(which == pair);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i) cor[t][i] = 0.f;
        for (int s = 0; s < cnt; ++s) {
          const __amdgpu_buffer_rsrc_t rb = stage_rsrc(s);
          A a;
          load_a(a, base, s);
#pragma unroll
          for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(
                  rb, ((w * 4 + (pair >> (2 * e) & 3)) * 2 + h) * row_bytes + j * 8, 0, 0);
#pragma unroll
              for (int t = 0; t < 2; ++t)
                cor[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x[e][w], __uint_as_float(x[t]), cor[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const bool mine = info[g * 32 + 8 * (i / 4) + 4 * h + i % 4].y == pair;
#pragma unroll
          for (int t = 0; t < 2; ++t)   // (every finite sum stays as it is, bit for bit)
            acc[t][i] = acc[t][i] * 0.f == 0.f || !mine ? acc[t][i] : cor[t][i];
        }
      }
    }
    uint32_t at[16];
    rows_at(at, g);
    if (whole && past) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (at[i] != kNone) __builtin_nontemporal_store(f32x2_s{acc[0][i], acc[1][i]}, reinterpret_cast<f32x2_any *>(place(at[i], uint32_t(8 * j))));
    } else if (whole) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (at[i] != kNone) *reinterpret_cast<f32x2_any *>(place(at[i], uint32_t(8 * j))) = f32x2_s{acc[0][i], acc[1][i]};
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (n0 + 2 * j + t < out_n)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (at[i] != kNone) *place(at[i], uint32_t(8 * j + 4 * t)) = acc[t][i];
    }
  }
}

}  // namespace

rbgp_reg_fn rbgp_reg_rows_kernel(int T, bool far) {
  if (T == 3) return far ? spmm_reg_rows<3, true> : spmm_reg_rows<3, false>;
  return far ? spmm_reg_rows<2, true> : spmm_reg_rows<2, false>;
}
