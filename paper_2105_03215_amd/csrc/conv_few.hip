// Implicit-GEMM convolution for few output pixels (an image network at batch 1 or
// a few): small tiles, the reduction split over the waves of a workgroup, MFMA
// operands straight from global memory.
//
// These layers are latency-bound: a 64x64 tiling leaves most of the chip idle,
// and its stage loop pays a load latency and a barrier every 64 elements;
// split over workgroups, a second launch adds the partial sums.  Here a tile
// is 16 or 32 pixels x 16 or 32 channels, so there are enough workgroups, and
// its four waves each take every fourth 64-element step of the reduction with no
// barrier and no LDS: U steps of loads are issued before the first MFMA that
// uses them, so a wave's share costs a load latency or two.  The waves' sums
// meet in LDS and are added in wave order (run-to-run identical); bias and residual
// are fetched before the reduction.  What is left is launch and prologue, about
// 4 us, and the operand bytes of a CU at about 40 GB/s (8 or 16 waves: no faster).
// us per layer in a chain, against split-K with its reduce launch: 3x3 256 ->
// 256 at 14x14 10.5 -> 7.7, 128 -> 128 at 28x28 10.2 -> 6.7; against four 4-wave groups
// on a 64x64 tile: 3x3 64 -> 64 at 56x56 8.2 -> 6.1.
//
// A step is 64 channels of one tap (Cp % 64 == 0): lane l reads 16 bytes at
// chunks l / 16 and 4 + l / 16 of row l % 16, so a row's 128-byte line is
// fetched once.  Weights are the MFMA A operand: a lane ends with 4
// consecutive channels of one pixel.
#include <type_traits>

#include "lds_dma.h"

namespace byoc {
namespace {

using namespace dma;

constexpr int kFewWaves = 4;

template <int TM, int TN>
__device__ __forceinline__ void conv_few_tile(ConvParams p) {
  constexpr int BM = TM * 16, BN = TN * 16, KG = kFewWaves;
  // steps in flight per wave (144 or 160 registers of operands): a 3x3 of 256
  // channels on 16x16 tiles is one batch of nine
  constexpr int U = TM + TN == 2 ? 9 : TM + TN == 3 ? 6 : 5;
  __shared__ f32x4 red[KG][TM * TN][64];
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
  constexpr int OPT = (kOut + 64 * KG - 1) / (64 * KG);  // per thread
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.res), (short)0, p.res ? p.res_bytes : 0, kBufferFlags);
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.bias), (short)0, p.bias ? ((p.Kp + 255) / 256) * 256 * 4 : 0, kBufferFlags);
  uint2 resv[OPT];
  f32x4 bv[OPT];
#pragma unroll
  for (int o = 0; o < OPT; ++o) {
    const int q = tid + o * 64 * KG;
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
  for (int t0 = wave; t0 < nst; t0 += KG * U) {
    uint4 a[U][TN][2], b[U][TM][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * KG;
      if (t >= nst) break;  // uniform per wave
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
    }
    __builtin_amdgcn_sched_barrier(0);  // every load of the U steps before the first MFMA
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (t0 + u * KG >= nst) break;  // uniform per wave
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[u][i][h]), as_bf16x8(b[u][j][h]),
                                                                acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) red[wave][i * TM + j][lane] = acc[i][j];
  lds_barrier();

  const ActClamp ac = act_clamp_of(p.act, p.alpha);
  auto finish = [&](auto mode_tag) {
    constexpr int G = decltype(mode_tag)::value;
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
      const int q = tid + o * 64 * KG;
      const int px = q / (BN / 4), ch = q % (BN / 4);  // pixel and group of 4 channels in the tile
      const int m = m0 + px, k = n0 + ch * 4;
      if (q >= kOut || m >= p.M || k >= p.Kp) continue;
      const int tile = (ch >> 2) * TM + (px >> 4), l = (ch & 3) * 16 + (px & 15);
      f32x4 v = red[0][tile][l];
#pragma unroll
      for (int w = 1; w < KG; ++w) v += red[w][tile][l];
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

template <int TM, int TN>
__global__ __launch_bounds__(64 * kFewWaves) void conv_few_kernel(ConvParams p) {
  conv_few_tile<TM, TN>(p);
}

// independent convs in one launch (blockIdx.y: the conv)
template <int TM, int TN>
__global__ __launch_bounds__(64 * kFewWaves) void grouped_conv_few_kernel(ConvGroup g) {
  const ConvParams p = g.p[blockIdx.y];
  if (outside_group_member<TM * 16, TN * 16>(p)) return;
  conv_few_tile<TM, TN>(p);
}

template <int TM, int TN>
hipError_t launch_group(ConvGroup& g, int n, hipStream_t s) {
  const dim3 grid = group_grid(g, n, TM * 16, TN * 16);
  grouped_conv_few_kernel<TM, TN><<<grid, 64 * kFewWaves, 0, s>>>(g);
  return hipGetLastError();
}

template <int TM, int TN>
hipError_t launch_one(const ConvParams& p_in, hipStream_t s) {
  ConvParams p = p_in;
  const int blocks = placed_blocks(p, TM * 16, TN * 16);
  conv_few_kernel<TM, TN><<<blocks, 64 * kFewWaves, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace

bool conv_few_ok(const ConvParams& p) { return p.Cp % 64 == 0 && p.R * p.S <= 32 && p.splits <= 1 && p.Kp % 4 == 0; }

hipError_t launch_conv_few_group(ConvGroup g, int n, int bm, int bn, hipStream_t s) {
  if (n < 1 || n > kConvGroup) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (!conv_few_ok(g.p[i])) return hipErrorInvalidValue;
  if (bm == 16 && bn == 16) return launch_group<1, 1>(g, n, s);
  if (bm == 16 && bn == 32) return launch_group<1, 2>(g, n, s);
  if (bm == 32 && bn == 16) return launch_group<2, 1>(g, n, s);
  if (bm == 32 && bn == 32) return launch_group<2, 2>(g, n, s);
  return hipErrorInvalidValue;
}

hipError_t launch_conv_few(const ConvParams& p, int bm, int bn, hipStream_t s) {
  if (!conv_few_ok(p)) return hipErrorInvalidValue;
  if (bm == 16 && bn == 16) return launch_one<1, 1>(p, s);
  if (bm == 16 && bn == 32) return launch_one<1, 2>(p, s);
  if (bm == 32 && bn == 16) return launch_one<2, 1>(p, s);
  if (bm == 32 && bn == 32) return launch_one<2, 2>(p, s);
  return hipErrorInvalidValue;
}

}  // namespace byoc
