// bf16 fused 3x3 convolution on the sparse matrix core, for masks whose tiles are 32 rows by 32 channels (|G_r.V| = 4,
// |G_i.V| = 8, the nine taps in G_b) and whose G_i keeps exactly one of the columns v and v + 4 (one 2-lift).  Of VGG19 with 128
// images, by the dispatch rule: forward layers 5, 7 at 1/4, 8 at 1/4 and 1/8, 9-11 at 1/4 to 1/16; input gradients of layers 3, 4 at
// 1/4, 5-7 at 1/4 and 1/8, 9-11 at 1/4 to 1/16.  (The rest have other tiles, few or the same tiles in
// a row, or fewer workgroups than CUs.)
//
// The register kernels load a channel nine times, once per tap, six of them at 2-byte alignment, and transpose it in
// registers.  Here a workgroup takes four rows of G_o x 32 T pixels in image order; the channels of the tiles that any of
// its rows has are loaded once, with the rows of pixels around them, and kept in LDS as an image [G_r vertex][pixel][8
// channels]: a tap is the same image read from another pixel, and eight channels of a pixel are the 16 bytes that a lane
// feeds the matrix core.  v_smfmac_f32_32x32x32_bf16 multiplies 32 rows x 32 pixels x 32 channels of one tap; a row keeps two of
// every four channels (columns 0, 4, 1, 5 and 2, 6, 3, 7 of G_i), which its index operand names.
// Weights: the lane of half h loads, of its row, stage h of the packed fragments (two G_r vertices, four kept channels, nine
// taps) with ten 16-byte loads, and pairs the channels of a tap with byte permutes whose selectors put the kept channel of
// column v mod 4 in place v: they depend on the row's G_i vertex only.
// A tile is summed by itself, its first five and its last four taps apart, and added to the total: the error against 64-bit
// sums is then that of the register kernels or less (VGG19 layer 9 at 1/4: 6.7e-8 against 9.2e-8; one chain 13e-8).
//
// us, register kernels -> this one: VGG19 conv3 at 8192 pixels 15.3 -> 13.6, its input gradient 16.7 -> 13.5, layer 6's at 32768
// pixels 53 -> 33; layer 9 at 1/8, 2048 pixels 14.6 -> 12.6, gradient 17.8 -> 12.7; the other sizes stand at the dispatch rule.
// What bounds it (conv3, timing-only builds of one chain): 13.6 in all, 9.5 without the products (launch 2.5; tables, channels
// and weights one after the other; stores 1), 11.2 without the staging, 12 without the reads of the image: one workgroup per CU
// has nothing to overlap these with, a larger batch has (16384 pixels: 19.3, not 28).
// Counters (conv3): matrix core 7 % busy, waves wait for 41 % of their cycles, LDS bank conflicts of 5000 cycles per CU (the stores
// of the image's pixels and their reads).
// Tried: fp32, operands split in three: layer 6 at 1/4, 8192 pixels 25.7 -> 29, its gradient 34.7 -> 29 (the one that gained), layer 9
// 25 -> 51 (three times the LDS: one or two tiles at once).  Stores that pair the bf16 sums of two lanes: 14.3 -> 16.9.
#include <hip/hip_runtime.h>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"
#include "rbgp_split.h"

using namespace rbgp_reg;
using namespace rbgp_split;

namespace {

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

template <int T>
__global__ __launch_bounds__(256, 2) void conv_tile(ConvTileParams p) {
  constexpr int NL = 10;
  extern __shared__ __attribute__((aligned(16))) u32x4 image[];   // [tile of the chunk][G_r vertex][pixel]
  const int lane = threadIdx.x & 63, h = lane >> 5, j = lane & 31;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), W = int(blockDim.x) >> 6;
  const int per = (p.a1 + W - 1) / W;           // workgroups of one column tile, all on XCD tile % 8
  const int slot = blockIdx.x >> 3, nt = int(blockIdx.x & 7) + 8 * (slot / per), ug = slot % per;
  if (nt >= p.ntiles) return;
  const int u1 = ug * W + wid;
  const bool has_row = u1 < p.a1;
  const uint64_t mine = has_row ? p.tiles[u1] : 0;
  uint64_t left = 0;                            // tile columns of the workgroup's rows that are still to come
  for (int w = 0; w < W; ++w) left |= ug * W + w < p.a1 ? p.tiles[ug * W + w] : 0;

  // the padded pixels from the row above the first pixel to the row below the last one (whole rows: W divides 32 T)
  auto center = [&](int n) {
    const int img = n / p.hw, r = n - img * p.hw, y = r / p.w, x = r - y * p.w;
    return (img * (p.h + 2) + y + 1) * p.w2 + x + 1;
  };
  const int n0 = nt * 32 * T, n_last = (n0 + 32 * T < p.n ? n0 + 32 * T : p.n) - 1;
  const int p_lo = center(n0) - p.w2 - 1, px = center(n_last) + p.w2 + 2 - p_lo;
  int at[T];                                    // the lane's pixel of every column block: bytes into a plane of the image
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int n = n0 + 32 * t + j;
    at[t] = (center(n < p.n ? n : n_last) - p_lo) * 16;
  }
  // the lane's row of a tile: G_i vertex and row of R
  const int ui = j / p.R, i = j - ui * p.R;
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

  f32x16 acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  const int plane = px * 16;                    // bytes
  u32x4 raw[NL];
  while (left) {
    uint64_t chunk = 0;                         // the next tiles, as many as LDS holds
    for (int k = 0; k < p.chunk && left; ++k) {
      chunk |= left & -left;
      left &= left - 1;
    }
    uint64_t own = mine & chunk;
    if (own) load_w(raw, __builtin_ctzll(own));
    // items of a tile x 64 lanes along the pixels, two pixels each; two items of 32 loads in flight per wave
    const int span = px >> 1, nq = (span + 63) >> 6, items = __popcll(chunk) * nq;   // (px is even)
    struct Item {
      int64_t x;
      int dst;                                  // -1: nothing
    };
    auto item = [&](int it) {
      const int k = it / nq, q = (it - k * nq) * 64 + lane;
      uint64_t c = chunk;
      for (int s = 0; s < k; ++s) c &= c - 1;
      return Item{int64_t(__builtin_ctzll(c) * 32) * p.chan + p_lo + 2 * (q < span ? q : 0), q < span ? k * 4 * px + 2 * q : -1};
    };
    for (int it = wid; it < items; it += 2 * W) {
      const bool two = it + W < items;
      const Item at2[2] = {item(it), item(two ? it + W : it)};
      uint32_t d[2][4][8];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int vr = 0; vr < 4; ++vr)
#pragma unroll
          for (int e = 0; e < 8; ++e)   // channels in the order 0, 4, 1, 5, 2, 6, 3, 7 of G_i's columns
            d[u][vr][e] = *reinterpret_cast<const uint32_t *>(static_cast<const uint16_t *>(p.X) + at2[u].x +
                                                              int64_t(vr * 8 + (e >> 1) + 4 * (e & 1)) * p.chan);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (at2[u].dst < 0 || (u == 1 && !two)) continue;
        u32x4 *const dst = image + at2[u].dst;
#pragma unroll
        for (int vr = 0; vr < 4; ++vr) {
          u32x4 lo, hi;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            lo[e] = __builtin_amdgcn_perm(d[u][vr][2 * e + 1], d[u][vr][2 * e], 0x05040100u);
            hi[e] = __builtin_amdgcn_perm(d[u][vr][2 * e + 1], d[u][vr][2 * e], 0x07060302u);
          }
          dst[vr * px] = lo;
          dst[vr * px + 1] = hi;
        }
      }
    }
    __syncthreads();
    while (own) {
      const int v = __builtin_ctzll(own);
      own &= own - 1;
      const int k = __popcll(chunk & ((uint64_t(1) << v) - 1));
      const unsigned char *img = reinterpret_cast<const unsigned char *>(image) + k * 4 * plane;
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
      f32x16 sum[2][T];                         // of this tile
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[0][t][e] = sum[1][t][e] = 0.f;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        if (tap == 4 && own) load_w(raw, __builtin_ctzll(own));   // (issued before the first tap: 0.7 us more)
        const int shift = ((tap / 3 - 1) * p.w2 + tap % 3 - 1) * 16 + h * plane;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const unsigned char *x = img + at[t] + shift;
          const bf16x16 b = joined(*reinterpret_cast<const u32x4 *>(x), *reinterpret_cast<const u32x4 *>(x + 2 * plane));
          sum[tap >= 5][t] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, a[tap]), b, sum[tap >= 5][t], sel.z, 0, 0);
        }
      }
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] += sum[0][t][e] + sum[1][t][e];
    }
    if (left) __syncthreads();
  }
  if (!has_row) return;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = 8 * (e / 4) + 4 * h + e % 4, rui = r / p.R, ri = r - rui * p.R;
    const int64_t m = ((int64_t(u1) * p.a2 + ri / p.a4) * p.a3 + rui) * p.a4 + ri % p.a4;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int n = n0 + 32 * t + j;
      if (n >= p.n) continue;
      if (p.obf16)
        __builtin_nontemporal_store(uint16_t(bf16_bits(acc[t][e])), reinterpret_cast<uint16_t *>(p.O) + m * p.ldO + n);
      else
        __builtin_nontemporal_store(acc[t][e], reinterpret_cast<float *>(p.O) + m * p.ldO + n);
    }
  }
}

}  // namespace

rbgp_conv_tile_fn rbgp_conv_tile_kernel(int T) { return T == 1 ? conv_tile<1> : T == 2 ? conv_tile<2> : nullptr; }
