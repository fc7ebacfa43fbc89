// The register family's kernel for few columns (spmm_reg in rbgp_mfma_reg.hip and spmm_reg_bf16 have the walk, the tables and the layouts):
// a workgroup is one (cluster, G_i vertex) pair on 16 columns, its stage list dealt to eight waves.
//
// Those kernels' waves take 64 columns, four waves at most a list: a batch of a few images leaves most CUs idle, and in fp32 a
// stage of 72 steps keeps the matrix core busy for 2304 cycles however few of the 64 columns exist.  Here a lane loads one column of
// its rows: v_mfma_f32_16x16x4 contracts the four lane groups' rows at once (576 cycles a stage), the bf16 rows need a shift and an or
// for two steps instead of a transposition, and the smaller operands leave room for eight waves of two stages in flight, two workgroups
// on a CU.  Partial sums meet in LDS and are added in one order; the error against 64-bit sums is 0.76 to 1.0 of spmm_reg's, in
// bf16 0.67 to 1.0.
//
// us, before -> this one, fp32, 512 x 4608: density 1/2, 16 columns fused 12.4 -> 5.9, 64 12.3 -> 7.8; 1/4 9.4 -> 4.9, 9.3 -> 5.6; 1/8,
// 128 columns 7.2 -> 4.6; its transpose at 1/4, four columns 5.6 -> 3.9; 256 x 2304 at 1/4, 64 to 256 columns 6.0 -> 4.1.  bf16: 1/2, 16
// columns fused 11.1 -> 4.7; 1/4, 64 8.4 -> 4.2; 1/8, 16 and 128 6.8 -> 4.0; 256 x 2304 at 1/2, 256 columns 7.4 -> 4.5.  What bounds it:
// a launch (2.7), the tables and the first stage's rows and weights, one memory latency after the other.  Tried: 16 waves a list, fp32,
// 16 columns 6.9 at 1/2 and 6.3 at 1/4 (starting them costs more than the stages they save).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rbgp_internal.h"
#include "rbgp_reg_common.h"

using namespace rbgp_reg;

namespace {

constexpr int W = 8;   // waves of a workgroup

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int KC, int RS, bool BF16>
__global__ __launch_bounds__(64 * W) void spmm_reg_narrow(RegParams p) {
  // rows of I and 16-byte loads of weights per lane and stage, bytes of one such load and of a fragment: as in spmm_reg, spmm_reg_bf16
  constexpr int NK32 = rbgp_bf16_blocks32(KC), ES = BF16 ? 2 : 4;
  constexpr bool TAIL = rbgp_bf16_tail16(KC);
  constexpr int MG = 16 / RS, NO = BF16 ? 8 * NK32 + (TAIL ? 4 : 0) : (KC + 3) / 4, NQ = BF16 ? NK32 + (TAIL ? 1 : 0) : (NO + 3) / 4;
  constexpr int QB = 4 * RS * 16, FB = NQ * QB;
  __shared__ float red[W][4][64];
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  table_args(p);
  WgCoord wg;
  if (!wg_coord(p, &wg)) return;
  const int cl = wg.cl, u3 = wg.u3, n0 = wg.ntq * 16;

  int mem[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm) mem[mm] = p.members[cl * MG + mm];
  const int32_t *rt = p.rowtab + u3 * (NO * 4);
  int off[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o)   // slot o of fp32: step 4 o + g; bf16: step o % 8 of the lane group's eight (four) of a block
    off[o] = rt[!BF16 ? o * 4 + g : o < 8 * NK32 ? o / 8 * 32 + 8 * g + o % 8 : NK32 * 32 + 4 * g + o % 8];
  // one of the wave's stages per lane: stage wid + lane * W of the list
  const int TS = p.tstride, own = wid + lane * W;
  const int32_t *stg = p.stages + int64_t(cl) * (1 + MG) * TS + (own < TS ? own : TS - 1);
  const int tb = stg[0];
  int tf[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm) tf[mm] = stg[(1 + mm) * TS];
  const int cnt0 = p.counts[cl], cnt = __builtin_amdgcn_readfirstlane(cnt0 > wid ? (cnt0 - wid + W - 1) / W : 0);
  // wave t < 4 adds up and stores row 4 g + t of the group
  const int i16 = 4 * g + (wid & 3), out_row = i16 % RS;
  const int out_u1 = p.members[cl * MG + i16 / RS], out_ofs = row_offset(p, u3, out_row);

  if (p.conv) {   // (spmm_reg: the entry of a group of four columns, two flags in its low bits)
    const int entry = p.colbase[(n0 + j) >> 2], first = (BF16 ? entry : entry & ~3) + (j & 3) * ES;
#pragma unroll
    for (int o = 0; o < NO; ++o) off[o] += first;
  } else {
#pragma unroll
    for (int o = 0; o < NO; ++o) off[o] = off[o] * (int(p.ldI) * ES) + j * ES;   // < 2^31: checked by the host
  }
  const uint32_t n0b = p.conv ? 0u : uint32_t(n0 * ES);
  const int mi = j / RS, alane = (g * RS + j % RS) * 16;
  const __amdgpu_buffer_rsrc_t rw =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.Wp), 0, p.w_bytes, kRsrcFlags);
  const int tbu = p.conv ? int(uint32_t(tb < 0 ? 0 : tb) / 9u) : (tb < 0 ? 0 : tb);   // first row (channel) of the stage
  const uint64_t i_first = reinterpret_cast<uint64_t>(p.I) + uint64_t(uint32_t(tbu)) * p.row_bytes + n0b;
  const int ib_lo = int(uint32_t(i_first)), ib_hi = int(uint32_t(i_first >> 32));
  const int rows_left = p.last_row - tbu < p.src_rows ? p.last_row - tbu : p.src_rows;
  const int ib_ext = tb >= 0 ? int(uint32_t(rows_left) * p.row_bytes + (p.n_bytes - n0b)) : 0;
  int aoff[MG];
#pragma unroll
  for (int mm = 0; mm < MG; ++mm)
    aoff[mm] = (tf[mm] >= 0 && mem[mm] >= 0) ? ((mem[mm] * p.fpm + tf[mm]) * p.a3 + u3) * FB : kOob;

  std::conditional_t<BF16, uint32_t, float> B[2][NO];
  f32x4 A[2][NQ], acc[4];   // of every fourth slot each (with two sums the error was up to a sixth above spmm_reg's)
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  // a stage past the wave's last one has extent zero and its weights past the buffer: zeros, no memory access
  auto stage_rows = [&](int s) {
    const int tl = s < 63 ? s : 63;
    const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_lo, tl))) |
                          (uint64_t(uint32_t(__builtin_amdgcn_readlane(ib_hi, tl))) << 32);
    const int ext = __builtin_amdgcn_readlane(ib_ext, tl);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, s < cnt ? ext : 0, kRsrcFlags);
  };
  auto stage_weights = [&](int s) {
    int addr = 0;
#pragma unroll
    for (int mm = 0; mm < MG; ++mm) {
      const int sv = __builtin_amdgcn_readlane(aoff[mm], s < 63 ? s : 63);
      addr = mi == mm ? sv : addr;
    }
    return (s < cnt ? addr : kOob) + alane;
  };
  auto load_row = [&](__amdgpu_buffer_rsrc_t r, int o) {
    if constexpr (BF16)
      return uint32_t(__builtin_amdgcn_raw_buffer_load_b16(r, off[o], 0, 0));
    else
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off[o], 0, 0));
  };
  auto fill = [&](int s, auto &b, f32x4 (&a)[NQ]) {
    const __amdgpu_buffer_rsrc_t r = stage_rows(s);
    const int av = stage_weights(s);
#pragma unroll
    for (int q = 0; q < NQ; ++q) a[q] = load_x4(rw, av, q * QB);
#pragma unroll
    for (int o = 0; o < NO; ++o) b[o] = load_row(r, o);
  };
  auto stage = [&](int s, auto &b, f32x4 (&a)[NQ]) {
    if constexpr (BF16) {
      auto two = [&](int o) { return b[o + 1] << 16 | b[o]; };
#pragma unroll
      for (int q = 0; q < NK32; ++q) {
        const u32x4 x = {two(8 * q), two(8 * q + 2), two(8 * q + 4), two(8 * q + 6)};
        acc[q & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[q]), __builtin_bit_cast(bf16x8, x), acc[q & 3], 0, 0, 0);
      }
      if constexpr (TAIL) {
        const u32x2 x = {two(8 * NK32), two(8 * NK32 + 2)}, w = {__float_as_uint(a[NK32][0]), __float_as_uint(a[NK32][1])};
        acc[NK32 & 3] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, w), __builtin_bit_cast(s16x4, x), acc[NK32 & 3], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int o = 0; o < NO; ++o) acc[o & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[o / 4][o % 4], b[o], acc[o & 3], 0, 0, 0);
    }
    if (s + 2 < cnt) fill(s + 2, b, a);
  };
  if (cnt > 0) {
    fill(0, B[0], A[0]);
    fill(1, B[1], A[1]);
    for (int s = 0; s < cnt; s += 2) {
      stage(s, B[0], A[0]);
      if (s + 1 < cnt) stage(s + 1, B[1], A[1]);
    }
  }

#pragma unroll
  for (int t = 0; t < 4; ++t) red[wid][t][lane] = (acc[0][t] + acc[1][t]) + (acc[2][t] + acc[3][t]);
  __syncthreads();
  if (wid >= 4) return;
  float sum[W];
#pragma unroll
  for (int k = 0; k < W; ++k) sum[k] = red[k][wid][lane];
  const float v = ((sum[0] + sum[1]) + (sum[2] + sum[3])) + ((sum[4] + sum[5]) + (sum[6] + sum[7]));
  if (out_u1 < 0 || out_row >= p.R || n0 + j >= p.N) return;
  const int64_t at = (int64_t(out_u1) * p.tm + u3 * p.a4 + out_ofs) * p.ldO + n0 + j;
  if (BF16 && p.obf16)
    reinterpret_cast<uint16_t *>(p.O)[at] = uint16_t(bf16_bits(v));
  else
    p.O[at] = v;
}

template <int KC, bool BF16>
rbgp_reg_fn by_rows(int RS) {
  return RS == 2 ? spmm_reg_narrow<KC, 2, BF16> : RS == 4 ? spmm_reg_narrow<KC, 4, BF16> : RS == 8 ? spmm_reg_narrow<KC, 8, BF16> : RS == 16 ? spmm_reg_narrow<KC, 16, BF16> : nullptr;
}

}  // namespace

rbgp_reg_fn rbgp_reg_narrow_kernel(int KC, int RS, bool bf16) {
  if (bf16) return KC == 72 ? by_rows<72, true>(RS) : KC == 36 ? by_rows<36, true>(RS) : KC == 32 ? by_rows<32, true>(RS) : KC == 18 ? by_rows<18, true>(RS) : nullptr;
  return KC == 72 ? by_rows<72, false>(RS) : KC == 36 ? by_rows<36, false>(RS) : KC == 32 ? by_rows<32, false>(RS) : KC == 18 ? by_rows<18, false>(RS) : nullptr;
}
