// Wave-split product for few tokens on gfx950: C^T = W * Act^T where a tiled
// kernel would leave most CUs idle or need split-K partials in memory and a
// second launch to add them.
//
// A workgroup of ks x FW waves owns FW x FI x 16 output features of TT x 16
// tokens.  Its ks wave rows each take a contiguous chunk of K, load both
// operands from memory straight into MFMA fragments (D 64-wide steps in flight,
// no LDS on the way) and leave their sums in LDS; after one barrier the waves
// add the ks partial sums in order (deterministic) and run the epilogue.  Bound by
// latency: what counts is the number of launches and the loads in flight.  The
// weights are read as a K-contiguous [features x K] matrix, so that nothing is
// laid out first.
//
// Measured against the tiled kernels with their reduces (whole calls, us): forward of 1B
// at 16 tokens 66 -> 25, at 64 68 -> 30, at 512 55 -> 49, of 350M at 2000 57 -> 40; training
// step of 350M at 1000 tokens 192 -> 96 (with the one launch of the weight gradients).
//
// The chunks are those of the tiled kernels' split-K, and within a chunk the sums
// run in the tiled kernels' order, so that the results are the same bits and a
// call's outputs do not depend on which of the two computes them.
//
// Fragment layout: of a 64-wide step, lane l takes of a dense operand row (feature
// or token) l % 16 at K 8 (l / 16) .. + 7 and 32 + 8 (l / 16) .. + 7.  Dense
// products take two v_mfma_f32_16x16x32_bf16, whose accumulators in lane l are
// features 4 (l / 16) .. + 3 of token l % 16: one whole group of 4 (Algorithm 1).
// A 2:4 operand is consumed by one v_smfmac_f32_16x16x64_bf16 (layout pinned by a
// probe: lane l holds the kept values of row l % 16 at dense K 16 (l / 16) .. + 15,
// its partner as above; the sums are those of two v_smfmac_f32_32x32x32_bf16 as the
// tiled kernel feeds them).  It must be the instruction's first operand, so there
// the accumulators are tokens 4 (l / 16) .. + 3 of feature l % 16.
#pragma once

#include "gemm.h"

namespace elas {

struct SmallArgs {
  const uint16_t* W;   // [features x K] weights, pitch ldw; rows >= m_valid and K entries >= kw_valid read as 0
  int64_t ldw;
  int m_valid, kw_valid;   // (dense tokens: kw_valid = K)
  int M, K;            // output features (SPARSIFY / DH: padded to 64) and contraction length
  int chunk, ks;       // 64-wide K steps per wave row, wave rows
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

// MAXW: the most waves it is launched with (ks x FW; 8 leave each wave 256 registers, 16 leave 128).
template <int EPI, bool SP, int TT, int FI, int FW, int D, int MAXW>
__global__ __launch_bounds__(64 * MAXW) void small_kernel(const SmallArgs g) {
  constexpr int FR = FI * TT;   // 16 x 16 blocks per wave
  extern __shared__ __attribute__((aligned(16))) f32x4 part[];   // [ks][FW * FR][64]
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ks = wave / FW, fw = wave % FW, nw = g.ks * FW;
  const int64_t t0 = (int64_t)blockIdx.y * (TT * 16);
  const int k_lane = lg * 8;                   // the lane's K offset in a step (and 32 more)
  const int f0 = (int)blockIdx.x * (FW * FI * 16) + fw * FI * 16;

  // (rows past the end re-read the last one; their results are not stored, or
  // zeroed where they are SPARSIFY's padding features)
  const uint16_t* wrow[FI];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int f = f0 + i * 16 + l16;
    wrow[i] = g.W + (int64_t)(f < g.m_valid ? f : g.m_valid - 1) * g.ldw + k_lane;
  }
  // (2:4: a workgroup's tokens lie in one block of 256 rows, R of which exist)
  const int64_t tb = t0 & ~(int64_t)255;
  const int R = (int)(g.T - tb < 256 ? g.T - tb : 256);
  const uint16_t* xrow[SP ? 1 : TT];
  uint32_t xoff[SP ? TT : 1], moff[SP ? TT : 1];
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int64_t t = t0 + j * 16 + l16 < g.T ? t0 + j * 16 + l16 : g.T - 1;
    if constexpr (SP) {
      xoff[j] = (uint32_t)((t - tb) * 32 + lg * 8);
      moff[j] = (uint32_t)((t - tb) * 8 + lg * 2);
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
        for (int i = 0; i < FI; ++i) a[d][i][h] = *(const uint4*)(wrow[i] + s * 64 + 32 * h);
        if constexpr (!SP) {
#pragma unroll
          for (int j = 0; j < TT; ++j) b[d][j][h] = *(const uint4*)(xrow[j] + s * 64 + 32 * h);
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < FI; ++i) a[d][i][h] = load16(wrow[i] + s * 64 + 32 * h, k + 32 * h < g.kw_valid);
        if constexpr (!SP) {
#pragma unroll
          for (int j = 0; j < TT; ++j) b[d][j][h] = load16(xrow[j] + s * 64 + 32 * h, k + 32 * h < g.kw_valid);
        }
      }
    }
    if constexpr (SP) {
      const uint16_t* xs = (const uint16_t*)uniform_ptr(g.X + tb * g.ldx + (int64_t)s * R * 32);
      const uint8_t* ms = (const uint8_t*)uniform_ptr(g.Xm + tb * g.ldxm + (int64_t)s * R * 8);
#pragma unroll
      for (int j = 0; j < TT; ++j) {
        b[d][j][0] = *(const uint4*)(xs + xoff[j]);
        m[d][j] = *(const uint16_t*)(ms + moff[j]);
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
        if constexpr (SP) {
#pragma unroll
          for (int i = 0; i < FI; ++i) {
            const bf16x16 w = __builtin_shufflevector(__builtin_bit_cast(bf16x8, a[d][i][0]), __builtin_bit_cast(bf16x8, a[d][i][1]),
                                                      0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
#pragma unroll
            for (int j = 0; j < TT; ++j)
              acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8, b[d][j][0]), w, acc[i][j], (int)m[d][j], 0, 0);
          }
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < TT; ++j)
#pragma unroll
              for (int i = 0; i < FI; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[d][i][h]),
                                                                    __builtin_bit_cast(bf16x8, b[d][j][h]), acc[i][j], 0, 0, 0);
        }
        if (s + D + d < s_end) load(s + D + d, d);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) part[((ks * FW + fw) * FR + i * TT + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  for (int q = wave; q < FW * FR; q += nw) {
    f32x4 c = part[q * 64 + lane];
    for (int k = 1; k < g.ks; ++k) c += part[(k * FW * FR + q) * 64 + lane];
    const int fb = (int)blockIdx.x * (FW * FI * 16) + (q / FR) * FI * 16 + (q % FR / TT) * 16;   // the block's first feature
    const int64_t t = t0 + (q % TT) * 16 + l16;
    if (fb >= g.M) continue;   // (uniform over the wave)
    const bool ok = t < g.T;
    if constexpr (SP) {
      // tokens 4 lg .. + 3 of feature fb + l16
      static_assert(EPI == EPI_BF16, "2:4 products: plain output");
      const int f = fb + l16;
      const int64_t ts = t0 + (q % TT) * 16 + 4 * lg;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f < g.M && ts + e < g.T) g.C[(ts + e) * g.ldc + f] = (uint16_t)bf16x2_rne(c[e], 0.f);
      continue;
    }
    if (EPI != EPI_BF16 && fb + 4 * lg >= g.m_valid) c = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == EPI_BF16) {
      const int f = fb + 4 * lg;
      if (ok && f < g.M) *(uint2*)(g.C + t * g.ldc + f) = make_uint2(bf16x2_rne(c[0], c[1]), bf16x2_rne(c[2], c[3]));
    } else {
      // group (fb % 64) / 4 + lg of the token's 64-feature entry block
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
