// Implicit-GEMM convolution for few output pixels (an image network at batch 1 or
// a few): small tiles, the reduction split over the waves of a workgroup, MFMA
// operands straight from global memory.
//
// These layers are latency-bound: a 64x64 tiling leaves most of the chip idle,
// and its stage loop pays a load latency and a barrier every 64 elements;
// split over workgroups, a second launch adds the partial sums.  Here a tile
// is 16 or 32 pixels x 16 or 32 channels, so there are enough workgroups, and
// its waves share the 64-element steps of the reduction with no barrier and
// no LDS: U steps of loads are issued before the first MFMA that uses them, so a
// wave's share costs a load latency or two.  Bias and residual are fetched before
// the reduction.  What is left is launch and prologue, about 4 us, and the
// operand bytes of a CU at about 40 GB/s.  us per layer in a chain of ten, replayed
// as a graph, against split-K with its reduce launch: 3x3 256 -> 256 at 14x14 11.0 -> 8.5,
// 128 -> 128 at 28x28 10.1 -> 7.4; against four 4-wave groups on a 64x64 tile:
// 3x3 64 -> 64 at 56x56 8.5 -> 6.7; against plain 64x64 tiles: 64 -> 64 at 28x28 4.6 -> 3.8.
//
// The sums are those of the plan that the layer would have without this kernel
// (few_segs, k_tiles_per_split), bit for bit: a segment is what one split of
// split-K or one reduction group sums in one accumulator - k_tiles_per_split
// consecutive steps, or (0) every few_segs-th step.  A wave takes whole segments
// and parks each one's sums in LDS, where they are added in segment order.
//
// A step is 64 channels of one tap (Cp % 64 == 0): lane l reads 16 bytes at
// chunks l / 16 and 4 + l / 16 of row l % 16, so a row's 128-byte line is
// fetched once.  Weights are the MFMA A operand: a lane ends with 4
// consecutive channels of one pixel.
#include <algorithm>
#include <type_traits>

#include "lds_dma.h"

namespace byoc {
namespace {

using namespace dma;

constexpr int kMaxSegs = 16;

template <int TM, int TN, int NW>
__device__ __forceinline__ void conv_few_tile(ConvParams p) {
  constexpr int BM = TM * 16, BN = TN * 16;
  // steps in flight per wave (144 or 160 registers of operands): a 3x3 of 256
  // channels on 16x16 tiles is one batch of nine
  constexpr int U = TM + TN == 2 ? 9 : TM + TN == 3 ? 6 : 5;
  extern __shared__ f32x4 red[];  // [few_segs][TM * TN][64]
  materialize_args(p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  if (!place_tile<BM, BN>(p, &tm, &tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  const int lr = lane & 15, lc = lane >> 4;
  const int PQ = p.P * p.Q;
  const int nst = p.Kg / 64;

  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.x), (short)0, p.x_bytes, kBufferFlags);
  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.w), (short)0, p.w_bytes, kBufferFlags);
  uint32_t woff[TN];
#pragma unroll
  for (int i = 0; i < TN; ++i) woff[i] = (uint32_t)(((n0 + i * 16 + lr) * p.Kgp + lc * 8) * 2);
  uint32_t xoff[TM], mask[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = m0 + j * 16 + lr;
    uint32_t bits = 0;
    int off = 0;
    if (m < p.M) {
      const int n = mdiv(m, p.mg_pq);
      const int pq = m - n * PQ;
      const int pp = mdiv(pq, p.mg_q);
      const int ih0 = pp * p.sh - p.pt;
      const int iw0 = (pq - pp * p.Q) * p.sw - p.pl;
      off = ((n * p.H + ih0) * p.W + iw0) * p.Cp + lc * 8;
      const int r_lo = max(0, -ih0), r_hi = min(p.R, p.H - ih0);
      const int s_lo = max(0, -iw0), s_hi = min(p.S, p.W - iw0);
      const uint32_t cols = s_hi > s_lo ? (uint32_t)(((1ull << s_hi) - 1ull) & ~((1ull << s_lo) - 1ull)) : 0u;
      for (int r = 0; r < p.R; ++r)
        if (r >= r_lo && r < r_hi) bits |= cols << (r * p.S);
    }
    xoff[j] = (uint32_t)off * 2u;
    mask[j] = bits;
  }

  // the outputs this thread finishes: 4 channels of a pixel
  constexpr int kOut = BM * BN / 4;                    // per tile
  constexpr int OPT = (kOut + 64 * NW - 1) / (64 * NW);  // per thread
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.res), (short)0, p.res ? p.res_bytes : 0, kBufferFlags);
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.bias), (short)0, p.bias ? ((p.Kp + 255) / 256) * 256 * 4 : 0, kBufferFlags);
  uint2 resv[OPT];
  f32x4 bv[OPT];
#pragma unroll
  for (int o = 0; o < OPT; ++o) {
    const int q = tid + o * 64 * NW;
    const int m = m0 + q / (BN / 4), k = n0 + q % (BN / 4) * 4;
    const bool ok = q < kOut && m < p.M && k < p.Kp;
    resv[o] = __builtin_bit_cast(
        uint2, __builtin_amdgcn_raw_buffer_load_b64(rr, ok ? (uint32_t)(m * p.ldr + k) * 2u : kOOB, 0, 0));
    bv[o] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(br, (uint32_t)k * 4u, 0, 0));
  }

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this wave's steps t0, t0 + step, ... below end; a segment is seg_len of them
  const int kps = p.k_tiles_per_split;
  const int spw = (p.few_segs + NW - 1) / NW;  // segments of a wave (1 where they are interleaved)
  const int step = kps > 0 ? 1 : p.few_segs;
  const int seg_len = kps > 0 ? kps : nst;
  const int end = kps > 0 ? min(nst, (wave + 1) * spw * kps) : wave < p.few_segs ? nst : 0;
  int seg = wave * spw, left = seg_len;
  for (int t0 = kps > 0 ? seg * kps : wave; t0 < end; t0 += step * U) {
    uint4 a[U][TN][2], b[U][TM][2];
    static_for<0, U>([&](auto u_tag) {
      constexpr int u = decltype(u_tag)::value;
      const int t = t0 + u * step;
      if (t >= end) return;  // uniform per wave
      const int rs = mdiv(t * 64, p.mg_cp);
      const int c = t * 64 - rs * p.Cp;
      const int r = mdiv(rs, p.mg_s);
      const uint32_t tap = (uint32_t)((r * p.W + rs - r * p.S) * p.Cp + c) * 2u;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
          a[u][i][h] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                     wr, woff[i] + t * 128u + h * 64u, 0, 0));
#pragma unroll
        for (int j = 0; j < TM; ++j)
          b[u][j][h] = __builtin_bit_cast(
              uint4, __builtin_amdgcn_raw_buffer_load_b128(
                         xr, (mask[j] >> rs) & 1u ? xoff[j] + tap + h * 64u : kOOB, 0, 0));
      }
    });
    __builtin_amdgcn_sched_barrier(0);  // every load of the U steps before the first MFMA
    static_for<0, U>([&](auto u_tag) {
      constexpr int u = decltype(u_tag)::value;
      const int t = t0 + u * step;
      if (t >= end) return;  // uniform per wave
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[u][i][h]), as_bf16x8(b[u][j][h]),
                                                                acc[i][j], 0, 0, 0);
      if (--left == 0 || t + step >= end) {  // the segment's last step
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j) {
            red[(seg * TM * TN + i * TM + j) * 64 + lane] = acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        ++seg;
        left = seg_len;
      }
    });
  }
  lds_barrier();

  const ActClamp ac = act_clamp_of(p.act, p.alpha);
  auto finish = [&](auto mode_tag) {
    constexpr int G = decltype(mode_tag)::value;
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
      const int q = tid + o * 64 * NW;
      const int px = q / (BN / 4), ch = q % (BN / 4);  // pixel and group of 4 channels in the tile
      const int m = m0 + px, k = n0 + ch * 4;
      if (q >= kOut || m >= p.M || k >= p.Kp) continue;
      const int tile = (ch >> 2) * TM + (px >> 4), l = (ch & 3) * 16 + (px & 15);
      f32x4 v = red[tile * 64 + l];
      for (int g = 1; g < p.few_segs; ++g) v += red[(g * TM * TN + tile) * 64 + l];
      const float rv[4] = {bf16_to_f32((bf16_t)(resv[o].x & 0xFFFF)), bf16_to_f32((bf16_t)(resv[o].x >> 16)),
                           bf16_to_f32((bf16_t)(resv[o].y & 0xFFFF)), bf16_to_f32((bf16_t)(resv[o].y >> 16))};
      float f[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = epilogue_value<G>(v[e] + bv[o][e], rv[e], ac);
      *(uint2*)(p.y + (size_t)m * p.ldy + k) = make_uint2(pack2_bf16(f[0], f[1]), pack2_bf16(f[2], f[3]));
    }
  };
  if (p.res_post)
    finish(std::integral_constant<int, 3>{});
  else if (act_mode(p.act) == 1)
    finish(std::integral_constant<int, 1>{});
  else
    finish(std::integral_constant<int, 0>{});
}

template <int TM, int TN, int NW>
__global__ __launch_bounds__(64 * NW) void conv_few_kernel(ConvParams p) {
  conv_few_tile<TM, TN, NW>(p);
}

// independent convs in one launch (blockIdx.y: the conv)
template <int TM, int TN, int NW>
__global__ __launch_bounds__(64 * NW) void grouped_conv_few_kernel(ConvGroup g) {
  const ConvParams p = g.p[blockIdx.y];
  if (outside_group_member<TM * 16, TN * 16>(p)) return;
  conv_few_tile<TM, TN, NW>(p);
}

// Waves for `segs` segments and that many workgroups per XCD: one per segment, up
// to eight while every workgroup has a CU to itself; eight leave room for no second
// one, so beyond that four with two segments or more each (192 -> 192 1x7 at
// 17x17, 5 segments, 30 workgroups per XCD: 9.9 us on eight waves, 8.9 on four).
int waves_of(int segs, int per_xcd) {
  return segs <= 1 ? 1 : segs <= 4 || per_xcd > kXcdSlots ? 4 : 8;
}

template <int TM, int TN, int NW>
hipError_t launch_waves(const ConvGroup& g, int n, int segs, dim3 grid, hipStream_t s) {
  const size_t lds = (size_t)segs * TM * TN * 64 * sizeof(f32x4);
  if (n == 1) conv_few_kernel<TM, TN, NW><<<grid, 64 * NW, lds, s>>>(g.p[0]);
  else grouped_conv_few_kernel<TM, TN, NW><<<grid, 64 * NW, lds, s>>>(g);
  return hipGetLastError();
}

// n convs on the same tile, with waves for the one of most segments
template <int TM, int TN>
hipError_t launch_tile(ConvGroup& g, int n, hipStream_t s) {
  const dim3 grid = n == 1 ? dim3(placed_blocks(g.p[0], TM * 16, TN * 16)) : group_grid(g, n, TM * 16, TN * 16);
  int segs = 1;
  for (int i = 0; i < n; ++i) segs = std::max(segs, g.p[i].few_segs);
  switch (waves_of(segs, (int)(grid.x + 7) / 8 * n)) {
    case 1: return launch_waves<TM, TN, 1>(g, n, segs, grid, s);
    case 4: return launch_waves<TM, TN, 4>(g, n, segs, grid, s);
    default: return launch_waves<TM, TN, 8>(g, n, segs, grid, s);
  }
}

}  // namespace

bool conv_few_ok(const ConvParams& p) {
  return p.Cp % 64 == 0 && p.R * p.S <= 32 && p.splits <= 1 && p.Kp % 4 == 0 && p.few_segs >= 1 &&
         p.few_segs <= kMaxSegs &&
         // every segment has a step: consecutive ones end at the last step, interleaved ones have a wave each
         (p.k_tiles_per_split > 0 ? (p.Kg / 64 + p.k_tiles_per_split - 1) / p.k_tiles_per_split == p.few_segs
                                  : p.few_segs <= 4 && p.few_segs <= p.Kg / 64);
}

int conv_few_waves(ConvParams p, int bm, int bn) { return waves_of(p.few_segs, (placed_blocks(p, bm, bn) + 7) / 8); }

hipError_t launch_conv_few_group(ConvGroup g, int n, int bm, int bn, hipStream_t s) {
  if (n < 1 || n > kConvGroup) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (!conv_few_ok(g.p[i])) return hipErrorInvalidValue;
  if (bm == 16 && bn == 16) return launch_tile<1, 1>(g, n, s);
  if (bm == 16 && bn == 32) return launch_tile<1, 2>(g, n, s);
  if (bm == 32 && bn == 16) return launch_tile<2, 1>(g, n, s);
  if (bm == 32 && bn == 32) return launch_tile<2, 2>(g, n, s);
  return hipErrorInvalidValue;
}

hipError_t launch_conv_few(const ConvParams& p, int bm, int bn, hipStream_t s) {
  ConvGroup g{};
  g.p[0] = p;
  return launch_conv_few_group(g, 1, bm, bn, s);
}

}  // namespace byoc
