// fp32 convolution (groups = 1) and dense layers of fp32 graphs on the fp32
// matrix cores: implicit GEMM over NCHW, true fp32 products and fp32
// accumulation (v_mfma_f32_16x16x4_f32).
//
// What bounds it: the MFMA rate (157 TFLOP/s) and the work around it.  A workgroup's
// stage is 32 * KG elements of the reduction, staged through LDS; between the
// MFMAs of two stages lie a barrier, the LDS reads and the issue of the input
// loads (4 bytes each along the pixels, a bounds select per element), so
// one workgroup per CU reaches half of the rate and two or three small tiles
// per CU hide each other's gaps.  The loads of PF stages are in flight in
// registers.  8 x 128 x 28 x 28 by 128 channels 3x3: 86 us on vector FMAs with
// scalar weights, 43 here; dense 300 x 768 x 2048 1989 -> 22, 30 rows 521 -> 8.4.
//
// M = output channels (weights [K][ldw], kk = (c*R + r)*S + s, zero padded), N =
// output pixels of all images.  LDS rows are kk-contiguous (stride + 4 floats: 8
// consecutive rows start on 8 different bank groups), so a lane takes 4 elements of its
// row per 16-byte read and the four MFMAs of 16 kk use element t of every
// lane - a permutation of kk common to both operands.
//
// KG wave groups share one tile's reduction (each takes 32 elements of every
// stage) where the tiles are too few to fill the chip; their sums meet in LDS
// in a fixed order.
#include "lds_dma.h"

namespace byoc {
namespace {

using dma::f32x4;
using dma::static_for;

// BM channels x BN pixels; WM x WN waves per reduction group.  ROWS: dense
// layers (a pixel's channels are contiguous), otherwise NCHW images.
template <int BM, int BN, int WM, int WN, int KG, bool ROWS, int PF>
__global__ __launch_bounds__(64 * WM * WN * KG) void conv_f32_mfma_kernel(ConvF32Params p) {
  constexpr int NT = 64 * WM * WN * KG;
  constexpr int BK = 32 * KG;
  constexpr int LD = BK + 4;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int AQ = BM * BK / 4 / NT, BQ = BN * BK / 4 / NT;  // 4-element groups per thread and stage
  static_assert(TM >= 1 && TN >= 1 && AQ >= 1 && BQ >= 1 && NT % BN == 0, "tile");
  __shared__ float lds[2][(BM + BN) * LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
  const int ntk = (p.K + BM - 1) / BM;
  const int tp = blockIdx.x / ntk, tk = blockIdx.x - tp * ntk;
  const int k0 = tk * BM, m0 = tp * BN;
  const int PQ = p.P * p.Q, M = p.N * PQ;
  const int CRS = p.C * p.R * p.S, HW = p.H * p.W;
  const int nst = (CRS + BK - 1) / BK;

  // operand groups of this thread: weight rows, and pixel tid % BN (ROWS:
  // pixel rows like the weight rows)
  const int aq = tid % (BK / 4), ar = tid / (BK / 4);  // kk group, first row
  constexpr int AROWS = NT / (BK / 4);                 // rows per pass
  const float* wa[AQ];  // (rows past the last channel repeat it and are not stored)
#pragma unroll
  for (int i = 0; i < AQ; ++i) wa[i] = p.w + (size_t)min(k0 + ar + i * AROWS, p.K - 1) * p.ldw + aq * 4;
  // Images: a lane keeps its pixel's window origin and a bit per tap inside the
  // image; the offsets and bits of a stage's elements come from the table one
  // stage before its loads are issued (as vector loads: scalar ones share a
  // counter with the LDS reads and stalled both).
  constexpr int BKQ = NT / BN;
  const int bkq = tid / BN;
  uint32_t xoff = 0, mask = 0;
  const __amdgpu_buffer_rsrc_t tr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<F32Tap*>(p.taps), (short)0, ROWS ? 0 : p.ldw * 8, kBufferFlags);
  uint4 lut[BQ][2];  // {offset, bit} of the 4 elements of each group of the next stage to load
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.x), (short)0, p.N * p.C * HW * 4, kBufferFlags);
  if constexpr (!ROWS) {
    const int m = m0 + tid % BN;
    if (m < M) {
      const int n = m / PQ, pq = m - n * PQ;
      const int pp = pq / p.Q;
      const int ih0 = pp * p.sh - p.pt, iw0 = (pq - pp * p.Q) * p.sw - p.pl;
      xoff = (uint32_t)(n * p.C * HW + ih0 * p.W + iw0) * 4u;  // (the tap's offset brings it into the buffer)
      for (int r = 0; r < p.R; ++r)
        for (int s = 0; s < p.S; ++s)
          if ((unsigned)(ih0 + r) < (unsigned)p.H && (unsigned)(iw0 + s) < (unsigned)p.W)
            mask |= 1u << (r * p.S + s);
    }
  }

  f32x4 ra[PF][AQ], rb[PF][BQ];
  auto look_up = [&](int st) {  // (past the table: zeros)
#pragma unroll
    for (int i = 0; i < BQ; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        lut[i][h] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(tr, (uint32_t)(st * BK + (bkq + i * BKQ) * 4 + 2 * h) * 8u, 0, 0));
  };
  auto load = [&](int st, auto set) {
    constexpr int U = decltype(set)::value;
    if (st >= nst) return;
    const int kb = st * BK;
#pragma unroll
    for (int i = 0; i < AQ; ++i) ra[U][i] = *(const f32x4*)(wa[i] + kb);
    if constexpr (ROWS) {
#pragma unroll
      for (int i = 0; i < BQ; ++i) {
        const int m = m0 + ar + i * AROWS, kk = kb + aq * 4;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (m < M) {
          const float* xr = p.x + (int64_t)m * p.C + kk;
          if (p.vec4) {
            if (kk < p.C) v = *(const f32x4*)xr;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (kk + e < p.C) v[e] = xr[e];
          }
        }
        rb[U][i] = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < BQ; ++i) {
        const uint32_t t[8] = {lut[i][0].x, lut[i][0].y, lut[i][0].z, lut[i][0].w,
                               lut[i][1].x, lut[i][1].y, lut[i][1].z, lut[i][1].w};
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                               xr, (mask & t[2 * e + 1]) != 0 ? xoff + t[2 * e] : kOOB, 0, 0));
        rb[U][i] = v;
      }
      look_up(st + 1);
    }
  };
  auto store = [&](int b, auto set) {
    constexpr int U = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < AQ; ++i) *(f32x4*)(&lds[b][(ar + i * AROWS) * LD + aq * 4]) = ra[U][i];
    if constexpr (ROWS) {
#pragma unroll
      for (int i = 0; i < BQ; ++i) *(f32x4*)(&lds[b][(BM + ar + i * AROWS) * LD + aq * 4]) = rb[U][i];
    } else {
#pragma unroll
      for (int i = 0; i < BQ; ++i) *(f32x4*)(&lds[b][(BM + tid % BN) * LD + (bkq + i * BKQ) * 4]) = rb[U][i];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int lr = lane & 15, lk = (lane >> 4) * 4 + kg * 32;
  // Operands of one stage: read after its barrier and before the next stage is
  // stored, so the stores and the following loads run behind the MFMAs.
  f32x4 fa[2][TM], fx[2][TN];
  auto read = [&](int b) {
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {  // 16 kk each
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[ch][i] = *(const f32x4*)(&lds[b][(wm * WTM + i * 16 + lr) * LD + lk + ch * 16]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fx[ch][j] = *(const f32x4*)(&lds[b][(BM + wn * WTN + j * 16 + lr) * LD + lk + ch * 16]);
    }
  };
  auto mma = [&] {
#pragma unroll
    for (int ch = 0; ch < 2; ++ch)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[ch][i][t], fx[ch][j][t], acc[i][j], 0, 0, 0);
  };

  // PF stages of loads in flight, stage st in register set st % PF (stages
  // past the end are not loaded)
  if constexpr (!ROWS) look_up(0);
  static_for<0, PF>([&](auto u) { load(decltype(u)::value, u); });
  store(0, std::integral_constant<int, 0>{});
  load(PF, std::integral_constant<int, 0>{});
  lds_barrier();
  for (int s0 = 0; s0 < nst; s0 += PF) {
    static_for<0, PF>([&](auto u) {
      const int st = s0 + decltype(u)::value;
      if (st >= nst) return;
      read(st & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (st + 1 < nst) {
        constexpr std::integral_constant<int, (decltype(u)::value + 1) % PF> set{};
        store((st + 1) & 1, set);  // (its last readers passed the barrier before this stage)
        load(st + 1 + PF, set);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma();
      lds_barrier();  // (a full fence would wait for the loads just issued)
    });
  }

  if constexpr (KG > 1) {  // the groups' sums, added in group order by group 0
    static_assert(KG * BM * BN <= 2 * (BM + BN) * LD, "reduction buffer");
    float* red = &lds[0][0];
    auto at = [&](int g, int i, int j) {
      return red + ((((g * WM * WN + wave % (WM * WN)) * TM + i) * TN + j) * 64 + lane) * 4;
    };
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4*)at(kg, i, j) = acc[i][j];
    }
    lds_barrier();
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] += *(const f32x4*)at(g, i, j);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int m = m0 + wn * WTN + j * 16 + lr;
    if (m >= M) continue;
    const int n = ROWS ? m : m / PQ, pq = ROWS ? 0 : m - n * PQ;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int kq = k0 + wm * WTM + i * 16 + 4 * (lane >> 4);
      if (ROWS && p.vec4_out) {  // (K % 4 == 0: the lane's four channels are all there or none)
        if (kq >= p.K) continue;
        const int64_t o = (int64_t)m * p.K + kq;
        f32x4 v = acc[i][j];
        if (p.bias) v += *(const f32x4*)(p.bias + kq);
        if (p.res) v += *(const f32x4*)(p.res + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], p.act, p.alpha);
        *(f32x4*)(p.y + o) = v;
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = kq + e;
        if (k >= p.K) continue;
        const int64_t o = ((int64_t)n * p.K + k) * PQ + pq;
        float v = acc[i][j][e];
        if (p.bias) v += p.bias[k];
        if (p.res) v += p.res[o];
        p.y[o] = apply_act(v, p.act, p.alpha);
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int KG, bool ROWS>
hipError_t launch_tile(const ConvF32Params& p, hipStream_t s) {
  const int64_t blocks = ((int64_t)p.N * p.P * p.Q + BN - 1) / BN * ((p.K + BM - 1) / BM);
  if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  constexpr int kGroups = (BM + BN) * 8 * KG / (64 * WM * WN * KG);
  conv_f32_mfma_kernel<BM, BN, WM, WN, KG, ROWS, (kGroups <= 6 ? 3 : 2)><<<(unsigned)blocks, 64 * WM * WN * KG, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace

bool conv_f32_mfma_ok(const ConvF32Params& p) {
  // a bit per tap; byte offsets of x and of a weight row within 31 bits
  return p.groups == 1 && p.R * p.S <= 32 && (int64_t)p.C * p.R * p.S < (int64_t(1) << 24) &&
         (int64_t)p.N * p.C * p.H * p.W < (int64_t(1) << 29) && (int64_t)p.N * p.P * p.Q < (int64_t(1) << 30);
}

hipError_t launch_conv_f32_mfma(const ConvF32Params& p_in, hipStream_t s) {
  ConvF32Params p = p_in;
  const int64_t M = (int64_t)p.N * p.P * p.Q;
  if (M == 0 || p.K == 0) return hipSuccess;
  if (!p.rows && !p.taps) return hipErrorInvalidValue;
  p.vec4 = p.C % 4 == 0 && (uintptr_t)p.x % 16 == 0;
  p.vec4_out = p.K % 4 == 0 && (uintptr_t)p.y % 16 == 0 && (uintptr_t)p.res % 16 == 0;
  // The smallest tiles that still make work for the whole chip once or
  // twice win (more workgroups per CU overlap), with the reduction shared by
  // more waves the fewer they are.  Images, us (32x64 | 32x32 KG 2 | 16x16 KG 4 | 16x16
  // KG 8): 32 x 24 x 56 x 56 3x3 34 | 43 | 68 | 104; 4 x 256 x 14 x 14 56 | 29 | 38 | 40;
  // 1 x 64 x 28 x 28 17 | 10.5 | 7.7 | 8.4; 1 x 256 x 7 x 7 55 | 28 | 16 | 15.  Dense,
  // rows x in x out (64x64 | 64x32 KG 2 | 32x32 KG 2 | 16x16 KG 8): 5000 x 192 x 768 28 | 37 |
  // 33 | 91; 1000 x 512 x 1500 35 | 29 | 34 | 55; 300 x 768 x 2048 37 | 28 | 22 | 33;
  // 30 x 768 x 3072 30 | 21 | 11 | 8.4.
  auto tiles = [&](int bm, int bn) { return (M + bn - 1) / bn * ((p.K + bm - 1) / bm); };
  if (p.rows) {
    if (tiles(64, 64) >= 600) return launch_tile<64, 64, 2, 2, 1, true>(p, s);
    if (tiles(64, 32) >= 400) return launch_tile<64, 32, 2, 1, 2, true>(p, s);
    if (tiles(32, 32) >= 200) return launch_tile<32, 32, 2, 2, 2, true>(p, s);
    return launch_tile<16, 16, 1, 1, 8, true>(p, s);
  }
  if (tiles(32, 64) >= 384) return launch_tile<32, 64, 2, 2, 1, false>(p, s);
  if (tiles(32, 32) >= 160) return launch_tile<32, 32, 2, 2, 2, false>(p, s);
  if (tiles(16, 16) >= 100) return launch_tile<16, 16, 1, 1, 4, false>(p, s);
  return launch_tile<16, 16, 1, 1, 8, false>(p, s);
}

}  // namespace byoc
