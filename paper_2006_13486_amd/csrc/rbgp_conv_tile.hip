// bf16 fused 3x3 convolution on the sparse matrix core, for masks whose tiles are 32 rows by 32 channels (|G_r.V| = 4,
// |G_i.V| = 8, the nine taps in G_b) and whose G_i keeps exactly one of the columns v and v + 4 (one 2-lift): of VGG19's layers
// with images of four rows and more most from layer 3 at 1/4 on, both ways, but for long lists and large tiles of few images (the rule
// stands at the dispatch).
//
// The register kernels load a channel nine times, once per tap, six of them at 2-byte alignment, and transpose it in
// registers.  Here a workgroup takes four rows of G_o x 32 T pixels in image order; the channels of the tiles that any of
// its rows has are loaded once (eight pixels of eight channels per thread, transposed with byte permutes), with the rows of
// pixels around them, and kept in LDS as an image [G_r vertex][pixel][8 channels]: a tap is the same image read from another
// pixel, and eight channels of a pixel are the 16 bytes that a lane feeds the matrix core.  v_smfmac_f32_32x32x32_bf16
// multiplies 32 rows x 32 pixels x 32 channels of one tap; a row keeps two of every four channels (columns 0, 4, 1, 5 and 2, 6,
// 3, 7 of G_i), which its index operand names.
// Weights: the lane of half h loads, of its row, stage h of the packed fragments (two G_r vertices, four kept channels, nine
// taps) with ten 16-byte loads, and pairs the channels of a tap with byte permutes whose selectors put the kept channel of
// column v mod 4 in place v: they depend on the row's G_i vertex only.
// A tile is summed by itself, its first five and its last four taps apart, and added to the total: the error against 64-bit
// sums is then that of the register kernels or less (VGG19 layer 9 at 1/4: 6.7e-8 against 9.2e-8; one chain 13e-8).
//
// us, VGG19 conv3 at 8192 pixels, both ways: register kernels 15.3 and 16.7, four waves that load two pixels of a channel at a
// time and pass the phases one after the other 13.5, this one 9.5 (10.1 with the tiles of a row looked up and dealt to the waves in the
// prologue and the weights loaded before the channels; 20 900 -> 19 400 cycles a wave); layer 9 at 1/8, 2048 pixels 14.6, 11.2, 8.3; the other sizes
// stand at the dispatch rule.  What bounds it: a chain of latencies (launch 2.5; tables 0.6; the channels, all of conv3's in one
// round of loads; their first use) and then issue: 1000 vector instructions and 800 cycles of products a wave, two waves a SIMD.
// Counters (conv3): waves wait for 44 % of their cycles (four waves 41, of a longer launch), matrix core 11 % busy, vector
// instructions 40 % of a SIMD's cycles, bank conflicts 3070 cycles per CU (3420 with lane j on pixel j, 36.3 -> 35.9 for the training
// step; planes an odd number of places apart, pixels in order and a wave's tasks over eight planes 2560, but its loads are
// then spread over more lines: 36.9).
// Tried: fp32, operands split in three: layer 6 at 1/4, 8192 pixels 25.7 -> 29, its gradient 34.7 -> 29 (the one that gained), layer 9
// 25 -> 51 (three times the LDS: one or two tiles at once).
#include <hip/hip_runtime.h>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"
#include "rbgp_split.h"

using namespace rbgp_reg;
using namespace rbgp_split;

namespace {

typedef u32x4 u32x4_u __attribute__((aligned(4)));

// where a lane's fragment of 72 steps holds channel ch (0..7) of its stage at a tap: 16-byte load and element
struct Place {
  int load, elem;
};
constexpr Place place(int ch, int tap) {
  const int s = 9 * ch + tap;
  return s < 64 ? Place{s / 8, s % 8} : Place{8 + (s - 64) / 4, (s - 64) % 4};
}
template <int E0, int E1>
__device__ __forceinline__ uint32_t two_halves(const u32x4 &x0, const u32x4 &x1) {
  return __builtin_amdgcn_perm(x1[E1 / 2], x0[E0 / 2], (E0 % 2 ? 0x0302u : 0x0100u) | (E1 % 2 ? 0x07060000u : 0x05040000u));
}

// Wave (r, s) multiplies, of row r of the workgroup's four rows of G_o, every S-th tile from the s-th on (S = 1, 2).
template <int T, int S>
__global__ __launch_bounds__(256 * S, 2 / S) void conv_tile(ConvTileParams p) {
  constexpr int NL = 10, kRows = 4;
  extern __shared__ __attribute__((aligned(16))) u32x4 image[];   // twice [tile of the chunk][G_r vertex][pixel]
  const int lane = threadIdx.x & 63, h = lane >> 5, j = lane & 31;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), wr = wid & (kRows - 1), ws = wid / kRows;
  const int per = (p.a1 + kRows - 1) / kRows;   // workgroups of one column tile, all on XCD tile % 8
  // (what the prologue reads of the kernel arguments, at once: see grid_args)
  asm volatile("" ::"s"(p.by_per.mul), "s"(p.by_per.shift), "s"(p.by_hw.mul), "s"(p.by_hw.shift), "s"(p.by_w.mul), "s"(p.by_w.shift),
               "s"(p.by_R.mul), "s"(p.by_R.shift), "s"(p.a1), "s"(p.ntiles), "s"(p.tiles), "s"(p.rows),
               "s"(p.sel), "s"(p.Wp), "s"(p.X), "s"(p.chan), "s"(p.n), "s"(p.h), "s"(p.w), "s"(p.w2), "s"(p.hw), "s"(p.R), "s"(p.RS),
               "s"(p.frag_bytes), "s"(p.a3), "s"(p.w_bytes), "s"(p.d1));
  const int slot = blockIdx.x >> 3, stripe = rbgp_fast::quotient(slot, p.by_per), nt = int(blockIdx.x & 7) + 8 * stripe, ug = slot - stripe * per;
  if (nt >= p.ntiles) return;
  const int u1 = ug * kRows + wr;
  // tile columns of the wave's row; those of the workgroup's rows still to come; those that are this wave's, in ascending order as the
  // chunks are (one load of five words: row by row behind their conditions, and dealt to the waves here, each waited for the last)
  const uint64_t *const tiles = p.tiles + ug * kRows;
  const uint64_t mine = tiles[wr];
  uint64_t left = tiles[0] | tiles[1] | tiles[2] | tiles[3], todo = S == 1 ? mine : tiles[(1 + ws) * p.rows + wr];
  static_assert(kRows == 4 && S <= 2, "the tables of the tiles");

  // the padded pixels from the row above the first pixel to the row below the last one (whole rows: W divides 32 T)
  auto center = [&](int n) {
    const int img = rbgp_fast::quotient(n, p.by_hw), r = n - img * p.hw, y = rbgp_fast::quotient(r, p.by_w), x = r - y * p.w;
    return (img * (p.h + 2) + y + 1) * p.w2 + x + 1;
  };
  const int n0 = nt * 32 * T, n_last = (n0 + 32 * T < p.n ? n0 + 32 * T : p.n) - 1;
  const int p_lo = center(n0) - p.w2 - 1, px = center(n_last) + p.w2 + 2 - p_lo;
  // Pixel q of a plane lies in place q ^ (q / 16) % 8 of its octet: the eight pixels that a lane stores and the runs of pixels
  // that neighbouring lanes read then fall on (nearly) different banks.  A 16-byte read takes the lanes 0-3, 12-15, 20-27 of a half at a
  // time, then the others: those hold 16 pixels in a row each.
  const int pixel = 16 * (__builtin_popcount(j >> 2) & 1) + 4 * (j >> 3) + (j & 3);   // the lane's of a column block
  const int plane8 = (px + 7) & ~7, plane = plane8 * 16;   // places, bytes
  auto place_of = [](int q) { return q ^ ((q >> 4) & 7); };
  int at[T];                                    // the lane's pixel of every column block, counted from p_lo
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int n = n0 + 32 * t + pixel;
    at[t] = center(n < p.n ? n : n_last) - p_lo;
  }
  // the lane's row of a tile: G_i vertex and row of R
  const int ui = rbgp_fast::quotient(j, p.by_R), i = j - ui * p.R;
  const int4 sel = p.sel[ui];                   // byte selectors of the channels in places 0, 1 and 2, 3; index operand
  const int wofs = (h * p.a3 + ui) * p.frag_bytes + i * 16;
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  auto load_w = [&](u32x4 (&r)[NL], int v) {
    const int jo = __popcll(mine & ((uint64_t(1) << v) - 1));   // (adjacency lists are ascending)
    const int base = (u1 * p.d1 + jo) * 2 * p.a3 * p.frag_bytes + wofs;
#pragma unroll
    for (int l = 0; l < NL; ++l) r[l] = __builtin_amdgcn_raw_buffer_load_b128(rw, base + l * p.RS * 16, 0, 0);
  };
  // One task per thread and chunk (p.chunk tiles): eight pixels of the eight channels of a (tile, G_r vertex).  The last task of
  // a plane ends with the plane (and repeats pixels of the one before it: nothing past the end of X is read).
  const int octets = plane8 >> 3;
  u32x4 d[8];
  int dst = -1, dst_px = 0;                     // plane of the task's pixels in a buffer, first of them; -1: no task
  auto take = [&]() {                           // the next tiles, as many as a buffer holds
    uint64_t c = 0;
    if (__popcll(left) <= p.chunk) {
      c = left;
      left = 0;
      return c;
    }
    for (int k = 0; k < p.chunk && left; ++k) {
      c |= left & -left;
      left &= left - 1;
    }
    return c;
  };
  auto fetch = [&](uint64_t chunk) {
    // (threadIdx.x + 1/2) / octets lies at least 1 / (2 octets) from a whole number, 2^-11 of it: far beyond the reciprocal's error
    const int pl = int((float(int(threadIdx.x)) + 0.5f) * __builtin_amdgcn_rcpf(float(octets))), q = int(threadIdx.x) - pl * octets, k = pl >> 2;
    dst = -1;
    if (k >= __popcll(chunk)) return;
    uint64_t c = chunk;
    for (int s = 0; s < k; ++s) c &= c - 1;
    dst = pl;
    dst_px = 8 * q < px - 8 ? 8 * q : px - 8;
    const uint16_t *x = static_cast<const uint16_t *>(p.X) + int64_t(__builtin_ctzll(c) * 32 + (pl & 3) * 8) * p.chan + p_lo + dst_px;
#pragma unroll
    for (int e = 0; e < 8; ++e)                 // channels in the order 0, 4, 1, 5, 2, 6, 3, 7 of G_i's columns
      d[e] = *reinterpret_cast<const u32x4_u *>(x + int64_t((e >> 1) + 4 * (e & 1)) * p.chan);
  };
  auto store = [&](int buf) {
    if (dst < 0) return;
    u32x4 *const to = image + (buf * p.chunk * 4 + dst) * plane8;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      u32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_perm(d[2 * e + 1][x / 2], d[2 * e][x / 2], x % 2 ? 0x07060302u : 0x05040100u);
      to[place_of(dst_px + x)] = v;
    }
  };

  f32x16 acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  u32x4 raw[NL];
  uint64_t chunk = take();
  fetch(chunk);                                 // (before the weights, which are wanted later: loads return in order)
  if (todo) load_w(raw, __builtin_ctzll(todo));
  store(0);
  __syncthreads();
  for (int buf = 0;; buf ^= 1) {
    const uint64_t here = chunk;
    chunk = take();
    if (chunk) fetch(chunk);
    while (todo & here) {
      const int v = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int k = __popcll(here & ((uint64_t(1) << v) - 1));
      const unsigned char *img = reinterpret_cast<const unsigned char *>(image) + (buf * p.chunk + k) * 4 * plane + h * plane;
      u32x4 a[9];
      static_for<0, 9>([&](auto tc) {
        constexpr int tap = decltype(tc)::value;
        static_for<0, 2>([&](auto vc) {
          constexpr int vv = decltype(vc)::value;
          constexpr Place a0 = place(4 * vv, tap), a1 = place(4 * vv + 1, tap), a2 = place(4 * vv + 2, tap), a3 = place(4 * vv + 3, tap);
          const uint32_t p01 = two_halves<a0.elem, a1.elem>(raw[a0.load], raw[a1.load]);
          const uint32_t p23 = two_halves<a2.elem, a3.elem>(raw[a2.load], raw[a3.load]);
          a[tap][2 * vv] = __builtin_amdgcn_perm(p23, p01, uint32_t(sel.x));
          a[tap][2 * vv + 1] = __builtin_amdgcn_perm(p23, p01, uint32_t(sel.y));
        });
      });
      // the lanes of half 0 hold G_r vertices 0 and 2, those of half 1 vertices 1 and 3 (first and second half of the lane's 16 steps)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        f32x16 sum[2];                          // of this tile: taps 0-4 and 5-8, in turn
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[0][e] = sum[1][e] = 0.f;
        static_for<0, 9>([&](auto kc) {
          constexpr int kk = decltype(kc)::value, late = kk % 2, tap = kk / 2 + 5 * late;
          if (t == T - 1 && kk == 4 && todo) load_w(raw, __builtin_ctzll(todo));
          const unsigned char *x = img + place_of(at[t] + (tap / 3 - 1) * p.w2 + tap % 3 - 1) * 16;
          const bf16x16 b = joined(*reinterpret_cast<const u32x4 *>(x), *reinterpret_cast<const u32x4 *>(x + 2 * plane));
          sum[late] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, a[tap]), b, sum[late], sel.z, 0, 0);
        });
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] += sum[0][e] + sum[1][e];
      }
    }
    if (!chunk) break;
    store(buf ^ 1);                             // (last read before the barrier that opened this round)
    __syncthreads();
  }

  // The waves of a row add their sums through LDS, which hands them on as rows of pixels: a thread stores eight at a time.
  __syncthreads();
  float *const red = reinterpret_cast<float *>(image);   // [s][r][row of the tile][pixel]
  constexpr int PX = 32 * T;
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int t = 0; t < T; ++t)
      red[((ws * kRows + wr) * 32 + 8 * (e / 4) + 4 * h + e % 4) * PX + 32 * t + pixel] = acc[t][e];
  __syncthreads();
  const int es = p.obf16 ? 2 : 4;
  const bool wide = (reinterpret_cast<uintptr_t>(p.O) | uintptr_t(p.ldO * es)) % 16 == 0;
#pragma unroll
  for (int u = 0; u < 2 * T / S; ++u) {
    const int it = u * 256 * S + int(threadIdx.x), row = it / (PX / 8), x = it % (PX / 8) * 8;   // 128 rows of PX / 8 pieces
    const int o1 = ug * kRows + row / 32, r = row % 32;
    if (o1 >= p.a1 || n0 + x >= p.n) continue;
    const f32x4 *s0 = reinterpret_cast<const f32x4 *>(red + row * PX + x), *s1 = s0 + kRows * 32 * PX / 4;
    f32x4 v[2] = {s0[0], s0[1]};
    if constexpr (S == 2) {
      v[0] += s1[0];
      v[1] += s1[1];
    }
    const int rui = rbgp_fast::quotient(r, p.by_R), ri = r - rui * p.R, ra = rbgp_fast::quotient(ri, p.by_a4);
    const int64_t o = (((int64_t(o1) * p.a2 + ra) * p.a3 + rui) * p.a4 + ri - ra * p.a4) * p.ldO + n0 + x;
    if (p.obf16) {
      uint16_t *const out = static_cast<uint16_t *>(p.O) + o;
      const u32x4 w = {bf16_pair(v[0][0], v[0][1]), bf16_pair(v[0][2], v[0][3]), bf16_pair(v[1][0], v[1][1]), bf16_pair(v[1][2], v[1][3])};
      if (wide && n0 + x + 8 <= p.n) {
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(out));
      } else {
        for (int e = 0; e < 8 && n0 + x + e < p.n; ++e) out[e] = uint16_t(w[e / 2] >> (16 * (e % 2)));
      }
    } else {
      float *const out = static_cast<float *>(p.O) + o;
      if (wide && n0 + x + 8 <= p.n) {
        __builtin_nontemporal_store(v[0], reinterpret_cast<f32x4 *>(out));
        __builtin_nontemporal_store(v[1], reinterpret_cast<f32x4 *>(out) + 1);
      } else {
        for (int e = 0; e < 8 && n0 + x + e < p.n; ++e) out[e] = v[e / 4][e % 4];
      }
    }
  }
}

}  // namespace

rbgp_conv_tile_fn rbgp_conv_tile_kernel(int T, int S) {
  if (T == 1) return S == 1 ? conv_tile<1, 1> : S == 2 ? conv_tile<1, 2> : nullptr;
  if (T == 2) return S == 1 ? conv_tile<2, 1> : S == 2 ? conv_tile<2, 2> : nullptr;
  return nullptr;
}
