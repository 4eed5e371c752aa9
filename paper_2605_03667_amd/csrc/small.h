// Wave-split product for few tokens on gfx950: C^T = W * Act^T where a tiled
// kernel would leave most CUs idle or need split-K partials in memory and a
// second launch to add them.
//
// A workgroup of KS x FW waves owns FW x FI x 16 output features of TT x 16
// tokens.  Its KS wave rows each take a contiguous chunk of K, load both
// operands from memory straight into MFMA fragments (D 64-wide steps in flight,
// no LDS on the way) and leave their sums in LDS; after one barrier the waves
// add the KS partial sums in order (deterministic) and run the epilogue.  Bound by
// latency: what counts is the number of launches and the loads in flight.  The
// weights are read as a K-contiguous [features x K] matrix, so that nothing is
// laid out first.
//
// Fragment layout (v_mfma_f32_16x16x32_bf16, two per step): lane l takes row
// (feature or token) l % 16 and, for MFMA h, the 8 K entries from 32 h + 8 (l / 16)
// of the step.  A 2:4 operand is read 16 bytes of kept values at a time, so
// there (in both operands) they are those from 16 (l / 16) + 8 h.  With dense
// operands and the chunks of a split-K tiled product the sums therefore run in
// the tiled kernel's order and the results are the same bits.  The accumulators
// of lane l are features 4 (l / 16) .. + 3 of token l % 16: one whole group of 4
// (Algorithm 1).
#pragma once

#include "gemm.h"

namespace elas {

struct SmallArgs {
  const uint16_t* W;   // [features x K] weights, pitch ldw; rows >= m_valid and K entries >= kw_valid read as 0
  int64_t ldw;
  int m_valid, kw_valid;   // (dense tokens: kw_valid = K)
  int M, K;            // output features (SPARSIFY / DH: padded to 64) and contraction length
  int chunk;           // 64-wide K steps per wave row
  const uint16_t* X;   // dense tokens [T x K], pitch ldx; or kept values of a 2:4 operand, tiled, pitch ldx
  const uint8_t* Xm;   // its metadata, tiled, pitch ldxm
  int64_t ldx, ldxm, T;
  uint16_t* C;         // EPI_BF16: [T x M], pitch ldc
  int64_t ldc;
  uint16_t* sv;        // compressed S, tiled: written (SPARSIFY) / read (DH)
  uint8_t* sm;
  int64_t ldv, ldm;
  uint16_t* dv;        // DH: kept values of dH, written
};

template <int EPI, bool SP, int TT, int FI, int KS, int FW, int D>
__global__ __launch_bounds__(64 * KS * FW) void small_kernel(const SmallArgs g) {
  constexpr int NW = KS * FW, FR = FI * TT;   // 16 x 16 blocks per wave
  __shared__ __attribute__((aligned(16))) f32x4 part[KS][FW * FR][64];
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ks = wave / FW, fw = wave % FW;
  const int64_t t0 = (int64_t)blockIdx.y * (TT * 16);
  const int k_lane = lg * (SP ? 16 : 8);       // the lane's K offset in a step, and from MFMA 0 to MFMA 1
  constexpr int k_half = SP ? 8 : 32;
  const int f0 = (int)blockIdx.x * (FW * FI * 16) + fw * FI * 16;

  // (rows past the end re-read the last one; their results are not stored, or
  // zeroed where they are SPARSIFY's padding features)
  const uint16_t* wrow[FI];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int f = f0 + i * 16 + l16;
    wrow[i] = g.W + (int64_t)(f < g.m_valid ? f : g.m_valid - 1) * g.ldw + k_lane;
  }
  const uint16_t* xrow[TT];
  const uint8_t* mrow[SP ? TT : 1];
  int xstep[SP ? TT : 1], mstep[SP ? TT : 1];
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int64_t t = t0 + j * 16 + l16 < g.T ? t0 + j * 16 + l16 : g.T - 1;
    if constexpr (SP) {
      const int64_t tb = t & ~(int64_t)255;
      const int R = (int)(g.T - tb < 256 ? g.T - tb : 256);
      xrow[j] = g.X + tb * g.ldx + (t - tb) * 32 + lg * 8;
      mrow[j] = g.Xm + tb * g.ldxm + (t - tb) * 8 + lg * 2;
      xstep[j] = R * 32;
      mstep[j] = R * 8;
    } else {
      xrow[j] = g.X + t * g.ldx + k_lane;
    }
  }
  uint4 a[D][FI][2], b[D][TT][SP ? 1 : 2];
  uint32_t m[D][SP ? TT : 1];
  // (only the last step of a K that is no multiple of 64 is masked)
  auto load16 = [](const uint16_t* p, bool ok) __attribute__((always_inline)) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (ok) v = *(const uint4*)p;
    return v;
  };
  auto load = [&](int s, int d) __attribute__((always_inline)) {
    const int k = s * 64 + k_lane;
    if (s * 64 + 64 <= g.kw_valid) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < FI; ++i) a[d][i][h] = *(const uint4*)(wrow[i] + s * 64 + k_half * h);
        if constexpr (!SP) {
#pragma unroll
          for (int j = 0; j < TT; ++j) b[d][j][h] = *(const uint4*)(xrow[j] + s * 64 + k_half * h);
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < FI; ++i) a[d][i][h] = load16(wrow[i] + s * 64 + k_half * h, k + k_half * h < g.kw_valid);
        if constexpr (!SP) {
#pragma unroll
          for (int j = 0; j < TT; ++j) b[d][j][h] = load16(xrow[j] + s * 64 + k_half * h, k + k_half * h < g.kw_valid);
        }
      }
    }
    if constexpr (SP) {
#pragma unroll
      for (int j = 0; j < TT; ++j) {
        b[d][j][0] = *(const uint4*)(xrow[j] + (int64_t)s * xstep[j]);
        m[d][j] = *(const uint16_t*)(mrow[j] + (int64_t)s * mstep[j]);
      }
    }
  };
  f32x4 acc[FI][TT];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int s_end = min((g.K + 63) / 64, (ks + 1) * g.chunk);
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (ks * g.chunk + d < s_end) load(ks * g.chunk + d, d);
  for (int s = ks * g.chunk; s < s_end; s += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (s + d < s_end) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < TT; ++j) {
            uint4 x;
            if constexpr (SP)
              x = h == 0 ? expand2(make_uint2(b[d][j][0].x, b[d][j][0].y), m[d][j] & 0xFFu)
                         : expand2(make_uint2(b[d][j][0].z, b[d][j][0].w), m[d][j] >> 8);
            else
              x = b[d][j][h];
#pragma unroll
            for (int i = 0; i < FI; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[d][i][h]),
                                                                  __builtin_bit_cast(bf16x8, x), acc[i][j], 0, 0, 0);
          }
        if (s + D + d < s_end) load(s + D + d, d);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) part[ks][fw * FR + i * TT + j][lane] = acc[i][j];
  __syncthreads();
  for (int q = wave; q < FW * FR; q += NW) {
    f32x4 c = part[0][q][lane];
#pragma unroll
    for (int k = 1; k < KS; ++k) c += part[k][q][lane];
    const int fb = (int)blockIdx.x * (FW * FI * 16) + (q / FR) * FI * 16 + (q % FR / TT) * 16;   // the block's first feature
    const int64_t t = t0 + (q % TT) * 16 + l16;
    if (fb >= g.M) continue;   // (uniform over the wave)
    const bool ok = t < g.T;
    if (EPI != EPI_BF16 && fb + 4 * lg >= g.m_valid) c = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == EPI_BF16) {
      const int f = fb + 4 * lg;
      if (ok && f < g.M) *(uint2*)(g.C + t * g.ldc + f) = make_uint2(bf16x2_rne(c[0], c[1]), bf16x2_rne(c[2], c[3]));
    } else {
      // group (fb % 64) / 4 + lg of the token's 64-feature entry block
      const int64_t tb = t & ~(int64_t)255;
      const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
      const int64_t iv = tb * g.ldv + (fb >> 6) * R * 32 + (t - tb) * 32 + (fb & 63) / 2 + 2 * lg;
      const int64_t im = tb * g.ldm + (fb >> 6) * R * 8 + (t - tb) * 8 + (fb & 63) / 8;
      if constexpr (EPI == EPI_SPARSIFY) {
        const uint32_t p01 = bf16x2_rne(relu_f32(c[0]), relu_f32(c[1])), p23 = bf16x2_rne(relu_f32(c[2]), relu_f32(c[3]));
        const Top2 k = top2_keys_hi(p01, p23);
        uint32_t w = (top2_code_xor15(k) ^ 0xFu) << (4 * lg);
        const float x = __builtin_bit_cast(float, k.first << 2), y = __builtin_bit_cast(float, k.second << 2);
        const auto s32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
        w = s32[0] | s32[1];
        const auto s16 = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        w = s16[0] | s16[1];   // the four codes of the 16 features
        if (ok) {
          *(uint32_t*)(g.sv + iv) = bf16x2_rne(x * x, y * y);
          if (lg == 0) *(uint16_t*)(g.sm + im) = (uint16_t)w;
        }
      } else {
        static_assert(EPI == EPI_DH, "epilogue mode");
        if (ok) {
          const uint32_t v = *(const uint32_t*)(g.sv + iv);
          const uint32_t w = *(const uint16_t*)(g.sm + im) >> (4 * lg);
          const uint32_t i0 = w & 3u, i1 = (w >> 2) & 3u;
          const float d0 = i0 == 0u ? c[0] : i0 == 1u ? c[1] : c[2];
          const float d1 = i1 == 1u ? c[1] : i1 == 2u ? c[2] : c[3];
          // relu(h) = bf16(sqrt(s)), exact
          const uint32_t rr = bf16x2_rne(sqrt_for_bf16(__builtin_bit_cast(float, v << 16)),
                                         sqrt_for_bf16(__builtin_bit_cast(float, v & 0xFFFF0000u)));
          *(uint32_t*)(g.dv + iv) = bf16x2_rne(d0 * 2.0f * __builtin_bit_cast(float, rr << 16),
                                               d1 * 2.0f * __builtin_bit_cast(float, rr & 0xFFFF0000u));
        }
      }
    }
  }
}

}  // namespace elas
