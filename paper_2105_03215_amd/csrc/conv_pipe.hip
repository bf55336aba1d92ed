// Implicit-GEMM convolution for large outputs: big tiles, operands streamed
// HBM->LDS as in conv_dma, MFMA operand registers prefetched one k-step
// ahead.
//
// What bounds these layers is the per-CU operand feed, not the matrix cores:
// a BM x BN tile fetches (BM + BN) * 128 bytes per 64-deep stage for
// BM * BN / 16 MFMA cycles per CU (a 64x64 tile 64 bytes per cycle, a
// 128x128 tile 32, a 256x256 tile 16 of the 36-56 that the L2 delivers
// per CU with both operands), so a tile here is as large as the grid can
// afford.  With one or two waves per SIMD nothing hides the LDS reads any more,
// so each wave holds the operands of two k-steps in registers: while the
// MFMAs of one k-step issue, the ds_reads of the next are in flight.
//
// Step of a stage t (64 reduction elements, two k-steps of 16x16x32):
//   read (t, 1)            MFMA (t, 0)
//   wait for the fills of stage t + 1 and for the reads; barrier
//   fill stage t + NS into the slot of stage t (whose last reads are done)
//   read (t + 1, 0)        MFMA (t, 1)
// One barrier per stage; NS - 1 stages are in flight across it.  Fills past
// the end read zeros from an out-of-range offset, so the waits are constants.
//
// The reduction runs in the same order as conv_dma's single-group tiles and
// the register-staged kernel (k-steps ascending, one accumulator per output),
// so all of them give the same bits; with slice_major the stages are taken
// slice by slice, all taps of a 64-channel slice in turn, which is conv_halo's
// order and gives its bits.
//
// Epilogue without LDS: the packed weight row behind MFMA row r of channel
// tile i is 32 (i / 2) + 8 (r / 4) + 4 (i % 2) + r % 4 of the wave's channels,
// so the accumulators of a pair of channel tiles hold 8 consecutive channels of
// one pixel: 16-byte residual loads and stores, 64 contiguous bytes per pixel
// and instruction, and no barrier after the loop.  LDS weight rows use the
// swizzle key (row & 3) | (row & 8) / 2, which keeps those row sets free
// of bank conflicts (8 consecutive lanes hold 8 different keys).
//
// int8 codes (I8): a 128-byte row holds 128 channels, the same two k-steps of
// v_mfma_i32_16x16x64_i8 per stage, exact int32 sums, and the int8 kernels'
// epilogue (8-byte stores; not on the 256x256 tile, where it spills).  6272 x
// 1024 x 256 with a residual, with events: 16.1 us on conv_i8's 128x64 tile, 11.9 on
// 128x128 here.
#include <type_traits>

#include "lds_dma.h"
#include "quant_epilogue.h"

namespace byoc {
namespace {

using namespace dma;

constexpr int kCH = 8;  // 16-byte chunks per LDS row

__device__ __forceinline__ f32x4 mma(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}
__device__ __forceinline__ i32x4 mma(uint4 a, uint4 b, i32x4 c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
}

template <int BM, int BN, int WM, int WN, int NS, bool I8>
__global__ __launch_bounds__(64 * WM * WN) void conv_pipe_kernel(QConvParams q) {
  const ConvParams& p = q.g;
  constexpr int ES = I8 ? 1 : 2;     // bytes per element
  constexpr int kBK = 128 / ES;      // reduction elements per stage
  using Acc = std::conditional_t<I8, i32x4, f32x4>;
  constexpr int kNT = 64 * WM * WN;
  constexpr int kRowsPerPass = kNT / kCH;  // rows one load instruction of every wave covers
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int AR = BM / kRowsPerPass, BR = BN / kRowsPerPass;
  static_assert(BM % kRowsPerPass == 0 && BN % kRowsPerPass == 0 && kRowsPerPass % 16 == 0, "fill shape");
  static_assert(WTM % 16 == 0 && WTN % 32 == 0, "wave tile: whole MFMA rows, pairs of channel tiles");
  constexpr int LPS = AR + BR;
  constexpr int STAGE = (BM + BN) * kCH;  // uint4 per stage
  static_assert(NS >= 2 && (NS - 1) * LPS <= 63, "vmcnt immediate");

  __shared__ uint4 ring[NS * STAGE];
  materialize_args(p);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int r0 = tid / kCH;  // first row this thread fills (8 rows per wave)
  // logical chunk it fetches: slot lane % 8 of row r0 (the keys of every later row it fills are the same)
  const int cva = (lane & 7) ^ (r0 & 7);
  const int cvb = (lane & 7) ^ ((r0 & 3) | ((r0 & 8) >> 1));

  int tm, tn;
  if (!place_tile<BM, BN>(p, &tm, &tn)) return;
  const int m0 = tm * BM;
  const int n0 = tn * BN;
  const int nst = p.Kg / kBK;  // (Cp is a multiple of it)

  // Activation rows of this thread: element offset of the row's window origin
  // plus its chunk; tapmask bit r*S+s set when that tap lies inside the image.
  int pix[AR];
  uint32_t tapmask[AR];
  const int PQ = p.P * p.Q;
#pragma unroll
  for (int i = 0; i < AR; ++i) {
    const int m = m0 + r0 + i * kRowsPerPass;
    uint32_t mask = 0;
    int off = 0;
    if (m < p.M) {
      const int n = mdiv(m, p.mg_pq);
      const int pq = m - n * PQ;
      const int pp = mdiv(pq, p.mg_q);
      const int ih0 = pp * p.sh - p.pt;
      const int iw0 = (pq - pp * p.Q) * p.sw - p.pl;
      off = ((n * p.H + ih0) * p.W + iw0) * p.Cp + cva * (16 / ES);
      const int r_lo = max(0, -ih0), r_hi = min(p.R, p.H - ih0);
      const int s_lo = max(0, -iw0), s_hi = min(p.S, p.W - iw0);
      const uint32_t cols = s_hi > s_lo ? (uint32_t)(((1ull << s_hi) - 1ull) & ~((1ull << s_lo) - 1ull)) : 0u;
      for (int r = 0; r < p.R; ++r)
        if (r >= r_lo && r < r_hi) mask |= cols << (r * p.S);
    }
    pix[i] = off;
    tapmask[i] = mask;
  }
  const i32x4 xr = buffer_rsrc(p.x, p.x_bytes);
  const i32x4 wr = buffer_rsrc(p.w, p.w_bytes);
  // (packed rows are padded to 256, every tile's channels among them or read as zeros past the buffer)
  uint32_t wvoff[BR];
#pragma unroll
  for (int i = 0; i < BR; ++i) wvoff[i] = (uint32_t)((n0 + r0 + i * kRowsPerPass) * p.Kgp * ES + cvb * 16);

  // Reduction position of the next stage to fill and its operand offsets;
  // fill<q> issues load q of that stage (all activation rows, then the weight
  // rows), advance() moves to the next one.
  const bool slice_major = p.slice_major != 0;
  int r = 0, s = 0, c = 0, issued = 0;
  auto fill = [&](int slot, auto q_tag) {
    constexpr int q = decltype(q_tag)::value;  // (load number)
    uint4* dst = ring + slot * STAGE;
    const bool live = issued < nst;
    if constexpr (q < AR) {
      const int tap = (r * p.W + s) * p.Cp + c;
      const int bit = (r * p.S + s) & 31;
      const uint32_t off = live && ((tapmask[q] >> bit) & 1u) ? (uint32_t)(pix[q] + tap) * ES : kOOB;
      lds_fill16(xr, __builtin_amdgcn_readfirstlane(lds_addr(dst + (q * kRowsPerPass + wave * 8) * kCH)), off);
    } else {
      constexpr int i = q - AR;
      lds_fill16(wr, __builtin_amdgcn_readfirstlane(lds_addr(dst + (BM + i * kRowsPerPass + wave * 8) * kCH)),
                 live ? wvoff[i] + (uint32_t)((r * p.S + s) * p.Cp + c) * ES : kOOB);
    }
  };
  auto advance = [&] {
    ++issued;
    // (one straight line of selects: with a branch here the compiler keeps the
    // position in scratch memory, which doubles the kernel's time)
    const int c1 = c + kBK;
    const bool step = slice_major || c1 == p.Cp;  // to the next tap
    const int s1 = step ? s + 1 : s;
    const bool wrap_s = s1 == p.S;
    const int r1 = wrap_s ? r + 1 : r;
    const bool wrap_r = slice_major && r1 == p.R;
    s = wrap_s ? 0 : s1;
    r = wrap_r ? 0 : r1;
    c = slice_major ? (wrap_r ? c1 : c) : (step ? 0 : c1);
  };

  Acc acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = Acc{0, 0, 0, 0};

  // LDS offsets (uint4) of this lane's operand rows at chunk 0 of k-step 0;
  // the slot of chunk ks * 4 + lane / 16 is that XOR the row's key
  const int lr = lane & 15, lc = lane >> 4;
  int arow[2], brow[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    arow[ks] = (wm * WTM + lr) * kCH + ((ks * 4 + lc) ^ (lr & 7));
    // row 8 (lr / 4) + lr % 4 (+ 4 for odd channel tiles, 32 per pair): key (row & 3) | (row & 8) / 2
    brow[ks] = (BM + wn * WTN + 8 * (lr >> 2) + (lr & 3)) * kCH + ((ks * 4 + lc) ^ ((lr & 3) | (lr & 4)));
  }
  struct Frags {
    uint4 a[TN], b[TM];
  };
  constexpr int NR = TN + TM;  // operand reads per k-step
  auto read1 = [&](Frags& f, int slot, auto ks_tag, auto q_tag) {
    constexpr int ks = decltype(ks_tag)::value, q = decltype(q_tag)::value;
    const uint4* st = ring + slot * STAGE;
    if constexpr (q < TN)
      f.a[q] = st[brow[ks] + ((q >> 1) * 32 + (q & 1) * 4) * kCH];
    else
      f.b[q - TN] = st[arow[ks] + (q - TN) * 16 * kCH];
  };
  // The MFMAs of one k-step from `cur`, with the operand reads of the next
  // k-step and (FILL) the fills of one stage spread between them: issued in
  // one burst, the reads of all waves would queue at the LDS with every
  // wave's MFMAs behind them.
  auto phase = [&](const Frags& cur, Frags& nxt, int rslot, auto ks_tag, int fslot, auto fill_tag) {
    constexpr bool FILL = decltype(fill_tag)::value;
    constexpr int RG = TM > 4 ? TM - 2 : TM;  // the reads go between the first RG groups of MFMAs
    static_for<0, TM>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
#pragma unroll
      for (int i = 0; i < TN; ++i)
        acc[i][j] = mma(cur.a[i], cur.b[j], acc[i][j]);
      static_for<0, NR>([&](auto q) {
        if constexpr (decltype(q)::value * RG / NR == j) read1(nxt, rslot, ks_tag, q);
      });
      if constexpr (FILL)
        static_for<0, LPS>([&](auto q) {
          if constexpr (decltype(q)::value * TM / LPS == j) fill(fslot, q);
        });
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  static_for<0, NS>([&](auto i) {
    static_for<0, LPS>([&](auto q) { fill(decltype(i)::value, q); });
    advance();
  });
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * LPS) : "memory");
  Frags f0, f1;
  constexpr std::integral_constant<int, 0> k0{};
  constexpr std::integral_constant<int, 1> k1{};
  static_for<0, NR>([&](auto q) { read1(f0, 0, k0, q); });
  int slot = 0;
  for (int t = 0; t < nst; ++t) {
    const int next = slot + 1 == NS ? 0 : slot + 1;
    phase(f0, f1, slot, k1, 0, std::false_type{});
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * LPS) : "memory");
    // (past the end the reads of the next stage find a zero-filled slot and are not used)
    phase(f1, f0, next, k0, slot, std::true_type{});
    advance();
    slot = next;
  }
  // every fill has landed before the workgroup's LDS is given away
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // Epilogue: lane = pixel lr of each pixel tile, channels 32 pr + 8 lc ... + 7
  if constexpr (I8) {
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(p.res), (short)0, p.res ? p.res_bytes : 0, kBufferFlags);
    const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(q.qch), (short)0, ((p.Kp + 255) / 256) * 256 * 8, kBufferFlags);
#pragma unroll
    for (int pr = 0; pr < TN / 2; ++pr) {
      const int k = n0 + wn * WTN + pr * 32 + lc * 8;
      const bool kok = k < p.Kp;
      int2 qc[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint4 u = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(br, (uint32_t)(k * 8 + e * 16), 0, 0));
        qc[2 * e] = make_int2((int)u.x, (int)u.y);
        qc[2 * e + 1] = make_int2((int)u.z, (int)u.w);
      }
      uint2 resv[TM];
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WTM + j * 16 + lr;
        resv[j] = p.res ? __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(
                              rr, kok && m < p.M ? (uint32_t)(m * p.ldr + k) : kOOB, 0, 0))
                        : make_uint2(0u, 0u);
      }
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WTM + j * 16 + lr;
        if (!kok || m >= p.M) continue;
        int a[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = acc[2 * pr + (e >> 2)][j][e & 3];
        *(uint2*)(reinterpret_cast<int8_t*>(p.y) + (size_t)m * p.ldy + k) = finish8_i8(a, qc, resv[j], q, m, k);
      }
    }
    return;
  } else {
  const ActClamp ac = act_clamp_of(p.act, p.alpha);
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.res), (short)0, p.res ? p.res_bytes : 0, kBufferFlags);
  const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.bias), (short)0, p.bias ? ((p.Kp + 255) / 256) * 256 * 4 : 0, kBufferFlags);
  auto epilogue = [&](auto mode_tag) {
    constexpr int G = decltype(mode_tag)::value;
#pragma unroll
    for (int pr = 0; pr < TN / 2; ++pr) {
      const int k = n0 + wn * WTN + pr * 32 + lc * 8;
      const bool kok = k < p.Kp;
      float bv[8];
      {
        const uint32_t bo = (uint32_t)k * 4u;
        const float4 b0 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(br, bo, 0, 0));
        const float4 b1 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(br, bo + 16u, 0, 0));
        bv[0] = b0.x; bv[1] = b0.y; bv[2] = b0.z; bv[3] = b0.w;
        bv[4] = b1.x; bv[5] = b1.y; bv[6] = b1.z; bv[7] = b1.w;
      }
      uint4 resv[TM];
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WTM + j * 16 + lr;
        resv[j] = p.res ? __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                              rr, kok && m < p.M ? (uint32_t)(m * p.ldr + k) * 2u : kOOB, 0, 0))
                        : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WTM + j * 16 + lr;
        float f[8], rv[8];
        unpack8(resv[j], rv);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          f[e] = epilogue_value<G>(acc[2 * pr + (e >> 2)][j][e & 3] + bv[e], rv[e], ac);
        if (kok && m < p.M) *(uint4*)(p.y + (size_t)m * p.ldy + k) = pack8(f);
      }
    }
  };
  if (p.res_post)
    epilogue(std::integral_constant<int, 3>{});
  else if (act_mode(p.act) == 1)
    epilogue(std::integral_constant<int, 1>{});
  else if (act_mode(p.act) == 0)
    epilogue(std::integral_constant<int, 0>{});
  else
    epilogue(std::integral_constant<int, 2>{});
  }
}

template <int BM, int BN, int WM, int WN, int NS, bool I8>
hipError_t launch_one(const QConvParams& q_in, hipStream_t s) {
  static_assert(NS * (BM + BN) * 128 <= kLdsLimit, "LDS");
  QConvParams q = q_in;
  const int blocks = placed_blocks(q.g, BM, BN);
  conv_pipe_kernel<BM, BN, WM, WN, NS, I8><<<blocks, 64 * WM * WN, 0, s>>>(q);
  return hipGetLastError();
}


// (bm, bn, waves along bm, waves along bn, ring stages)
#define BYOC_PIPE_TILES(X) \
  X(256, 256, 2, 4, 2)     \
  X(256, 128, 4, 2, 3)     \
  X(128, 256, 2, 4, 3)     \
  X(128, 192, 4, 2, 3)     \
  X(128, 128, 2, 4, 2)     \
  X(128, 64, 2, 2, 3)      \
  X(64, 128, 2, 2, 3)      \
  X(64, 64, 2, 2, 3)

template <bool I8>
hipError_t launch_any(const QConvParams& q, int bm, int bn, int stages, int threads, hipStream_t s) {
  if (!conv_pipe_ok(q.g, I8)) return hipErrorInvalidValue;
#define X(M, N, A, B, S) \
  if constexpr (!I8 || M * N < 256 * 256)   \
    if (bm == M && bn == N && stages == S && threads == 64 * A * B) return launch_one<M, N, A, B, S, I8>(q, s);
  BYOC_PIPE_TILES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace

bool conv_pipe_ok(const ConvParams& p, bool i8) {
  return p.Cp % (i8 ? 128 : 64) == 0 && p.R * p.S <= 32 && p.splits <= 1;
}

bool conv_pipe_tile_supported(int bm, int bn, int stages, int threads) {
#define X(M, N, A, B, S) \
  if (bm == M && bn == N && stages == S && threads == 64 * A * B) return true;
  BYOC_PIPE_TILES(X)
#undef X
  return false;
}

hipError_t launch_conv_pipe(const ConvParams& p, int bm, int bn, int stages, int threads, hipStream_t s) {
  QConvParams q{};
  q.g = p;
  return launch_any<false>(q, bm, bn, stages, threads, s);
}

hipError_t launch_conv_pipe_i8(const QConvParams& q, int bm, int bn, int stages, int threads, hipStream_t s) {
  return launch_any<true>(q, bm, bn, stages, threads, s);
}

}  // namespace byoc
