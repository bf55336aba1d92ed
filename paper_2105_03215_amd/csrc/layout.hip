// Boundary layout transforms of 4-D tensors: NCHW (bf16 or f32, the caller's
// layout) to and from NHWC bf16 or int8 codes, the dtype conversion fused in.
//
// HBM-bound: both sides have to move in long runs, and they run along
// different axes.  A workgroup takes PT pixels x GT channel groups (16 bytes of
// one pixel each: 8 bf16 or 16 codes) through LDS: the NCHW side moves along the
// pixels (PX consecutive pixels per lane, 8- or 16-byte accesses), the NHWC
// side along the channels (GT lanes per pixel, GT * 16 contiguous bytes).  Writing
// each group straight from registers, as the kernels for narrow or tiny images
// do, puts 16-byte pieces Cp * 2 bytes apart.  With events around the launch
// (about 4 us of them its own cost): 16 x 128 x 56 x 56 bf16 to NHWC 17.0 -> 8.9 us,
// 32 x 512 x 28 x 28 bf16 to codes 21.7 -> 14.1, 32 x 1024 x 14 x 14 codes to f32
// 24.5 -> 7.9.
//
// LDS row of pixel p: slot g at g ^ key, key = (p ^ (p / 4)) % GT, so that
// consecutive lanes (pixels 4 apart, or 1 apart without vectors) use distinct
// banks.
#include "device_common.h"

namespace byoc {
namespace {

constexpr int kThreads = 256;

struct LayoutParams {
  const void* x;
  void* y;
  int C, HW, Cp;
  int ptiles, gtiles;  // tiles along the pixels of an image and along its channel groups
  float scale;         // quantize: fl32(1 / S); dequantize: fl32(S)
  int zp;
};

__device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ float to_f32(float v) { return v; }
template <class T>
__device__ __forceinline__ T from_f32(float v) {
  if constexpr (sizeof(T) == 2) return f32_to_bf16(v);
  else return v;
}

// (rint(v / S) clamped to [lo, hi] = [-128 - zp, 127 - zp]) + zp + 128; NaN gives code -128.
__device__ __forceinline__ float quantize_u8(float v, float inv, float lo, float hi, float off) {
  return fminf(fmaxf(rintf(v * inv), lo), hi) + off;
}

// The tile of this workgroup: image, first pixel, first channel group.
template <int PT, int GT>
__device__ __forceinline__ void tile_of(const LayoutParams& p, int* n, int* p0, int* g0) {
  const int b = (int)blockIdx.x;
  const int pg = b / p.gtiles;  // (channel tiles of one pixel run are neighbours)
  *g0 = (b - pg * p.gtiles) * GT;
  *n = pg / p.ptiles;
  *p0 = (pg - *n * p.ptiles) * PT;
}

template <int GT>
__device__ __forceinline__ int slot_of(int px, int g) {
  return px * GT + (g ^ ((px ^ (px >> 2)) & (GT - 1)));
}

// VEC: HW % 4 == 0 and x aligned to 4 elements, PX == 4.
template <class SrcT, bool CODES, int GT, int PX, bool VEC>
__global__ __launch_bounds__(kThreads) void to_nhwc_kernel(LayoutParams p) {
  constexpr int CH = CODES ? 16 : 8;       // channels of a group
  constexpr int LN = kThreads / GT;        // lanes along the pixels
  constexpr int PT = LN * PX;
  struct alignas(sizeof(SrcT) * PX) Vec {
    SrcT e[PX];
  };
  __shared__ uint4 tile[PT * GT];
  int n, p0, g0;
  tile_of<PT, GT>(p, &n, &p0, &g0);
  const int q = threadIdx.x % LN, g = threadIdx.x / LN;
  const int c0 = (g0 + g) * CH;
  const SrcT* x = (const SrcT*)p.x + ((size_t)n * p.C + c0) * p.HW;
  auto pixel = [&](int i) { return VEC ? q * PX + i : q + LN * i; };
  if (c0 < p.Cp) {
    SrcT v[CH][PX];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const bool cok = c0 + c < p.C;
      if constexpr (VEC) {
        Vec u{};
        if (cok && p0 + q * PX < p.HW) u = *(const Vec*)(x + (size_t)c * p.HW + p0 + q * PX);
#pragma unroll
        for (int i = 0; i < PX; ++i) v[c][i] = u.e[i];
      } else {
#pragma unroll
        for (int i = 0; i < PX; ++i) {
          const int px = p0 + pixel(i);
          v[c][i] = cok && px < p.HW ? x[(size_t)c * p.HW + px] : SrcT(0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < PX; ++i) {
      uint32_t w[4];
      if constexpr (CODES) {
        const float lo = (float)(-128 - p.zp), hi = (float)(127 - p.zp), off = (float)(p.zp + 128);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          w[j] = kU8ToCode;  // channels past C: code 0
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (c0 + 4 * j + c < p.C) w[j] = put_u8(quantize_u8(to_f32(v[4 * j + c][i]), p.scale, lo, hi, off), c, w[j]);
          w[j] ^= kU8ToCode;
        }
      } else if constexpr (sizeof(SrcT) == 2) {
#pragma unroll
        for (int c = 0; c < CH; c += 2) w[c >> 1] = (uint32_t)v[c][i] | ((uint32_t)v[c + 1][i] << 16);
      } else {
#pragma unroll
        for (int c = 0; c < CH; c += 2) w[c >> 1] = pack2_bf16(v[c][i], v[c + 1][i]);
      }
      tile[slot_of<GT>(pixel(i), g)] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
  __syncthreads();
  char* y = (char*)p.y + ((size_t)n * p.HW + p0) * p.Cp * (16 / CH);
#pragma unroll
  for (int t = 0; t < PT * GT / kThreads; ++t) {
    const int k = t * kThreads + threadIdx.x, px = k / GT, gg = k % GT;
    if (p0 + px < p.HW && (g0 + gg) * CH < p.Cp)
      *(uint4*)(y + (size_t)px * p.Cp * (16 / CH) + (g0 + gg) * 16) = tile[slot_of<GT>(px, gg)];
  }
}

// VEC: HW % 4 == 0 and y aligned to 4 elements, PX == 4.
template <class DstT, bool CODES, int GT, int PX, bool VEC>
__global__ __launch_bounds__(kThreads) void to_nchw_kernel(LayoutParams p) {
  constexpr int CH = CODES ? 16 : 8;
  constexpr int LN = kThreads / GT;
  constexpr int PT = LN * PX;
  struct alignas(sizeof(DstT) * PX) Vec {
    DstT e[PX];
  };
  __shared__ uint4 tile[PT * GT];
  int n, p0, g0;
  tile_of<PT, GT>(p, &n, &p0, &g0);
  const char* x = (const char*)p.x + ((size_t)n * p.HW + p0) * p.Cp * (16 / CH);
#pragma unroll
  for (int t = 0; t < PT * GT / kThreads; ++t) {
    const int k = t * kThreads + threadIdx.x, px = k / GT, gg = k % GT;
    if (p0 + px < p.HW && (g0 + gg) * CH < p.Cp)
      tile[slot_of<GT>(px, gg)] = *(const uint4*)(x + (size_t)px * p.Cp * (16 / CH) + (g0 + gg) * 16);
  }
  __syncthreads();
  const int q = threadIdx.x % LN, g = threadIdx.x / LN;
  const int c0 = (g0 + g) * CH;
  if (c0 >= p.C) return;
  auto pixel = [&](int i) { return VEC ? q * PX + i : q + LN * i; };
  uint32_t w[PX][4];
#pragma unroll
  for (int i = 0; i < PX; ++i) {
    const uint4 u = tile[slot_of<GT>(pixel(i), g)];
    w[i][0] = u.x, w[i][1] = u.y, w[i][2] = u.z, w[i][3] = u.w;
  }
  DstT* y = (DstT*)p.y + ((size_t)n * p.C + c0) * p.HW;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    Vec o;
#pragma unroll
    for (int i = 0; i < PX; ++i) {
      if constexpr (CODES) {
        const int code = (int)(int8_t)(w[i][c >> 2] >> (8 * (c & 3)));
        o.e[i] = from_f32<DstT>(p.scale * (float)(code - p.zp));
      } else {
        const bf16_t h = (bf16_t)(w[i][c >> 1] >> (16 * (c & 1)));
        if constexpr (sizeof(DstT) == 2) o.e[i] = h;
        else o.e[i] = bf16_to_f32(h);
      }
    }
    const bool cok = c0 + c < p.C;
    if constexpr (VEC) {
      if (cok && p0 + q * PX < p.HW) *(Vec*)(y + (size_t)c * p.HW + p0 + q * PX) = o;
    } else {
#pragma unroll
      for (int i = 0; i < PX; ++i)
        if (cok && p0 + pixel(i) < p.HW) y[(size_t)c * p.HW + p0 + pixel(i)] = o.e[i];
    }
  }
}

// TO: towards NHWC; T: the element of the NCHW side.
template <bool TO, class T, bool CODES, int GT, int PX, bool VEC>
void launch_one(LayoutParams p, int64_t N, hipStream_t s) {
  constexpr int PT = kThreads / GT * PX;
  const int G = p.Cp / (CODES ? 16 : 8);
  p.ptiles = (p.HW + PT - 1) / PT;
  p.gtiles = (G + GT - 1) / GT;
  const unsigned blocks = (unsigned)(N * p.ptiles * p.gtiles);
  if constexpr (TO) to_nhwc_kernel<T, CODES, GT, PX, VEC><<<blocks, kThreads, 0, s>>>(p);
  else to_nchw_kernel<T, CODES, GT, PX, VEC><<<blocks, kThreads, 0, s>>>(p);
}

template <bool TO, class T, bool CODES, int GT>
void launch_gt(const LayoutParams& p, int64_t N, hipStream_t s) {
  const int G = p.Cp / (CODES ? 16 : 8);
  const void* nchw = TO ? p.x : p.y;
  constexpr int kPt4 = kThreads / GT * 4;
  const int64_t blocks4 = N * ((p.HW + kPt4 - 1) / kPt4) * ((G + GT - 1) / GT);
  // four pixels per lane where that still gives two workgroups per CU, or one
  // (64 x 56 x 56, one image: 25 workgroups become 98)
  if (blocks4 < 512)
    launch_one<TO, T, CODES, GT, 1, false>(p, N, s);
  else if (p.HW % 4 == 0 && (uintptr_t)nchw % (4 * sizeof(T)) == 0)
    launch_one<TO, T, CODES, GT, 4, true>(p, N, s);
  else
    launch_one<TO, T, CODES, GT, 4, false>(p, N, s);
}

template <bool TO, class T, bool CODES>
void launch_any(const LayoutParams& p, int64_t N, hipStream_t s) {
  // 8 groups (128 bytes of a pixel) per tile, or 4 where that leaves fewer groups idle
  const int G = p.Cp / (CODES ? 16 : 8);
  if ((G + 7) / 8 * 8 > (G + 3) / 4 * 4) launch_gt<TO, T, CODES, 4>(p, N, s);
  else launch_gt<TO, T, CODES, 8>(p, N, s);
}

}  // namespace

bool layout_tiled(int64_t N, int C, int64_t HW, int Cp, bool codes) {
  const int G = Cp / (codes ? 16 : 8);
  // at least two channel groups per pixel and 16 pixels per plane: below, the
  // per-group kernels already write (one group) or read (tiny planes) whole runs
  return G >= 2 && HW >= 16 && C <= Cp && N * HW * Cp < (int64_t(1) << 38) && HW < (int64_t(1) << 30) &&
         N * ((HW + 31) / 32) * ((G + 3) / 4) < (int64_t(1) << 31);
}

hipError_t launch_layout(const void* x, void* y, bool to_nhwc, bool bf16, bool codes, int N, int C, int HW, int Cp,
                         float scale, int zp, hipStream_t s) {
  LayoutParams p{x, y, C, HW, Cp, 0, 0, scale, zp};
  if (to_nhwc) {
    if (bf16) codes ? launch_any<true, bf16_t, true>(p, N, s) : launch_any<true, bf16_t, false>(p, N, s);
    else codes ? launch_any<true, float, true>(p, N, s) : launch_any<true, float, false>(p, N, s);
  } else {
    if (bf16) codes ? launch_any<false, bf16_t, true>(p, N, s) : launch_any<false, bf16_t, false>(p, N, s);
    else codes ? launch_any<false, float, true>(p, N, s) : launch_any<false, float, false>(p, N, s);
  }
  return hipGetLastError();
}

}  // namespace byoc
