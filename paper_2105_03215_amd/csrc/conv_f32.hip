// fp32 convolution on the vector ALU, for what the matrix-core kernel does not
// take (grouped convs, more than 32 taps, inputs of 2 GiB and more) and for images
// of many pixels with few output channels: direct
// NCHW evaluation of the conv composite, one thread per output, fused multiply-adds in fp32 over the
// reduction in (c, r, s) order, then bias, residual, activation.  Dense runs
// as the 1x1 case on [M, K, 1, 1]; consecutive threads take
// consecutive output columns so input rows are read contiguously.
#include <algorithm>

#include "device_common.h"

namespace byoc {
namespace {

__global__ __launch_bounds__(256) void conv_f32_kernel(ConvF32Params p) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = (int64_t)p.N * p.K * p.P * p.Q;
  if (idx >= total) return;
  const int q = (int)(idx % p.Q);
  int64_t t = idx / p.Q;
  const int pp = (int)(t % p.P);
  t /= p.P;
  const int k = (int)(t % p.K);
  const int n = (int)(t / p.K);
  const int cg = p.C / p.groups;
  const int kg = p.K / p.groups;
  const int g = k / kg;
  const int ih0 = pp * p.sh - p.pt;
  const int iw0 = q * p.sw - p.pl;
  float acc = 0.f;
  for (int c = 0; c < cg; ++c) {
    const float* xc = p.x + ((size_t)n * p.C + g * cg + c) * p.H * p.W;
    const float* wc = p.w + ((size_t)k * cg + c) * p.R * p.S;
    for (int r = 0; r < p.R; ++r) {
      const int ih = ih0 + r;
      if ((unsigned)ih >= (unsigned)p.H) continue;
      for (int s = 0; s < p.S; ++s) {
        const int iw = iw0 + s;
        if ((unsigned)iw >= (unsigned)p.W) continue;
        acc = fmaf(xc[ih * p.W + iw], wc[r * p.S + s], acc);
      }
    }
  }
  if (p.bias) acc += p.bias[k];
  if (p.res) acc += p.res[idx];
  p.y[idx] = apply_act(acc, p.act, p.alpha);
}

// Register-blocked form for groups == 1 and RxS taps known at compile
// time: one thread per output pixel computes KB output channels; the
// channel block is uniform over the workgroup (grid y), so its weights come
// through scalar loads shared by the wave, and the taps of two input
// channels are loaded at once.  Each output sums its terms in the order of
// the kernel above - channel, kernel row, column - from zero (a tap outside
// the image adds an exact zero), then bias, residual and activation.
constexpr int kKB = 4;

template <int R, int S>
__global__ __launch_bounds__(64) void conv_f32_regs_kernel(ConvF32Params p) {
  const int nkb = (p.K + kKB - 1) / kKB;
  const int n = blockIdx.y / nkb;
  const int k0 = (blockIdx.y - n * nkb) * kKB;
  const int pix = blockIdx.x * 64 + threadIdx.x;
  const bool live = pix < p.P * p.Q;
  const int pp = live ? pix / p.Q : 0;
  const int q = live ? pix - pp * p.Q : 0;
  const int ih0 = pp * p.sh - p.pt, iw0 = q * p.sw - p.pl;
  const int HW = p.H * p.W;
  // taps inside the image (offsets within a channel plane)
  int off[R * S];
  bool in[R * S];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < S; ++t) {
      const int ih = ih0 + r, iw = iw0 + t;
      in[r * S + t] = live && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      off[r * S + t] = in[r * S + t] ? ih * p.W + iw : 0;
    }
  const float* xn = p.x + (size_t)n * p.C * HW;
  const float* wk[kKB];
#pragma unroll
  for (int j = 0; j < kKB; ++j) wk[j] = p.w + (size_t)min(k0 + j, p.K - 1) * p.C * R * S;
  float acc[kKB];
#pragma unroll
  for (int j = 0; j < kKB; ++j) acc[j] = 0.f;
  auto tap_sum = [&](int c, const float* xv) {
#pragma unroll
    for (int t = 0; t < R * S; ++t)
#pragma unroll
      for (int j = 0; j < kKB; ++j) acc[j] = fmaf(xv[t], wk[j][c * R * S + t], acc[j]);
  };
  int c = 0;
  for (; c + 2 <= p.C; c += 2) {
    float xa[R * S], xb[R * S];
    const float* xc = xn + (size_t)c * HW;
#pragma unroll
    for (int t = 0; t < R * S; ++t) {
      xa[t] = in[t] ? xc[off[t]] : 0.f;
      xb[t] = in[t] ? xc[HW + off[t]] : 0.f;
    }
    tap_sum(c, xa);
    tap_sum(c + 1, xb);
  }
  if (c < p.C) {
    float xa[R * S];
    const float* xc = xn + (size_t)c * HW;
#pragma unroll
    for (int t = 0; t < R * S; ++t) xa[t] = in[t] ? xc[off[t]] : 0.f;
    tap_sum(c, xa);
  }
  if (!live) return;
#pragma unroll
  for (int j = 0; j < kKB; ++j) {
    const int k = k0 + j;
    if (k >= p.K) break;
    const size_t o = (((size_t)n * p.K + k) * p.P + pp) * p.Q + q;
    float v = acc[j];
    if (p.bias) v += p.bias[k];
    if (p.res) v += p.res[o];
    p.y[o] = apply_act(v, p.act, p.alpha);
  }
}

bool regs_ok(const ConvF32Params& p) {
  return p.groups == 1 && (int64_t)p.N * ((p.K + kKB - 1) / kKB) <= 65535 && (int64_t)p.P * p.Q < (int64_t(1) << 30) &&
         (int64_t)p.C * p.H * p.W < (int64_t(1) << 31) && p.R == p.S && (p.R == 3 || p.R == 1);
}

}  // namespace

// The matrix-core kernel's tile for many pixels has 32 channels, all of which it
// pays for, and takes the reduction in stages of 32: with few output channels or a short
// reduction the kernels above are faster.  The modelled times are us per million
// pixels on MI355X, plus a part per input channel or tap (their serial chain of loads) and
// per stage.  With events around the launch, measured (modelled) here | on the matrix cores,
// 16 x 224 x 224 3x3: 3 -> 1 11.7 (17.0) | 51.7 (51.6), 3 -> 16 42.2 (42.4) | 69.7 (70.8), 3 -> 32 79.1
// (79.8) | 74.7 (74.7); 16 -> 16 117 (125) | 144 (144); 32 -> 16 228 (227) | 225 (217); 1x1: 32 -> 8
// 37.5 (38.6) | 62.4 (68.8); 5x5: 1 -> 4 47.4 (59.3) | 75.3 (67.8); 2 x 112 x 112 3x3:
// 8 -> 8 6.7 (7.4) | 8.5 (8.9).  Fewer pixels than the rule asks for run on smaller
// matrix-core tiles, which were never slower by more than 1 us.
bool conv_f32_vector_faster(const ConvF32Params& p) {
  const double pix = (double)p.N * p.P * p.Q, crs = (double)p.C * p.R * p.S;
  if (p.groups != 1 || p.rows || pix < 64 * 384 || p.K > 64) return false;
  const int st = (int)((crs + 31) / 32), kg = std::min(p.K, 32);
  const double mfma =
      4.0 + 0.6 * st + pix * 1e-6 * ((p.K + 31) / 32) * (30.0 + 6.7 * std::min(kg, 4) + 0.3 * std::max(kg - 4, 0) + 22.0 * st);
  if (!regs_ok(p)) return 4.5 + 0.04 * crs + pix * 1e-6 * (p.K + 0.4) * (1.5 + 0.55 * crs) < mfma;
  const double mpix = p.N * (((int64_t)p.P * p.Q + 63) / 64 * 64e-6);  // (64-pixel blocks of an image)
  const double k4 = (p.K + kKB - 1) / kKB * kKB;
  return (p.R == 3 ? 4.3 + (0.26 + 0.002 * p.C) * p.C + mpix * std::max(6.0 + 0.33 * crs, k4 * (1.5 + 0.052 * crs))
                   : 4.3 + 0.075 * p.C + mpix * std::max(5.0 + 0.6 * crs, k4 * (1.4 + 0.11 * crs))) < mfma;
}

hipError_t launch_conv_f32(const ConvF32Params& p, hipStream_t s) {
  const int64_t total = (int64_t)p.N * p.K * p.P * p.Q;
  if (total == 0) return hipSuccess;
  if (regs_ok(p)) {
    const dim3 grid((unsigned)(((int64_t)p.P * p.Q + 63) / 64), (unsigned)(p.N * ((p.K + kKB - 1) / kKB)));
    if (p.R == 3) conv_f32_regs_kernel<3, 3><<<grid, 64, 0, s>>>(p);
    else conv_f32_regs_kernel<1, 1><<<grid, 64, 0, s>>>(p);
    return hipGetLastError();
  }
  conv_f32_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace byoc
