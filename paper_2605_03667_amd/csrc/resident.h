// Token-resident product for gfx950: C^T = W * Act^T for a short contraction
// (K = r = 128, 256 or 512): the up projection, dS and the two products back to
// the model width.
//
// A workgroup copies a block of 128 tokens (128 x K bf16, at most 128 KB) to
// LDS once and then runs over the output features.  Each wave takes blocks of
// 64 features on its own: their weights come straight from L2 into registers
// (the factor is laid out in MFMA fragment order, frag_index, so that every
// load is one contiguous KB), one 64-wide K panel ahead, and the tokens'
// fragments from LDS.  Nothing in the loop is shared for writing, so it has no
// barrier: the two waves of a SIMD drift apart and one wave's epilogue (vector
// ALU and stores, issued at a raised priority: 4 to 8 % on the up projection)
// runs under the other's MFMAs.  In a tiled kernel with K = 512 all eight waves
// reach the epilogue together, a third of its time.
//
// What bounds it is power: on dense bf16 MFMAs of random data the chip runs at
// 1.4 to 1.8 GHz, and the vector ALU work under them lowers it further.  The
// 16x16x32 MFMA is used because it draws less than the 32x32x16 (a loop of
// register operands alone: 1.87 against 1.59 PFLOP/s; the up projection at 1B
// and 65536 tokens 302 against 323 us).
//
// Measured at 1B, 65536 tokens, against the 256 x 256 tiled kernel of gemm.h:
// up projection with 2:4 selection 424 -> 307 us, masked dH 478 -> 334, Y
// 149 -> 137, dx 158 -> 138; 350M: 145 -> 103, 175 -> 112, 53 -> 49, 56 -> 49.
#pragma once

#include "gemm.h"

namespace elas {

// Fragment order of a K-contiguous factor [M x K] (K a multiple of 64, M padded
// to 64 rows) for v_mfma_f32_16x16x32_bf16: per 64-row block and 64-wide K
// panel 8 KB, in which the 1 KB of (k32 step, 16-row quarter i) holds lane l's
// 8 elements at 16 l bytes: row 16 i + l % 16, k 32 kk + 8 (l / 16) ...
// kp = K / 64.  Index of element (row, k).
__host__ __device__ inline int64_t frag_index(int64_t row, int64_t k, int64_t kp) {
  return ((row >> 6) * kp + (k >> 6)) * 4096 + ((k >> 5) & 1) * 2048 + ((row >> 4) & 3) * 512 + ((k >> 3) & 3) * 128 +
         (row & 15) * 8 + (k & 7);
}

// (global pointers, so that stores through a uniform base are not flat)
typedef __attribute__((address_space(1))) u32x4 gu32x4;
typedef __attribute__((address_space(1))) u32x2 gu32x2;

struct ResArgs {
  const uint16_t* W;   // frag_index layout, nfb blocks of 64 features
  const uint16_t* X;   // tokens [T x K], pitch ldx
  int64_t ldx, T;
  int nfb;             // blocks of 64 features
  int fsplit;          // workgroups per token block, each an equal share of the features
  // EPI_SPARSIFY (written) / EPI_DH (read): compressed S, tiled
  uint16_t* sv;
  uint8_t* sm;
  int64_t ldv, ldm;
  uint16_t* dv;        // EPI_DH: kept values of dH, tiled
  // Dense output [T x features], features < f_valid (a multiple of 8):
  // EPI_BF16 the product, EPI_ACT_DENSE relu(.)^2, EPI_DH_DENSE the product
  // times 2 relu(h) with s = relu(h)^2 read from act (same shape).
  uint16_t* C;
  const uint16_t* act;
  int64_t ldc, ld_act;
  int f_valid;
};

// v[i] of lane group lg (16 lanes) -> v[lg] of lane group i.
__device__ __forceinline__ void transpose4(uint32_t (&v)[4]) {
  const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  v[0] = c[0]; v[1] = c[1]; v[2] = d[0]; v[3] = d[1];
}

template <class F>
__device__ __forceinline__ void unroll8(F&& f) {
  f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{}); f(std::integral_constant<int, 2>{});
  f(std::integral_constant<int, 3>{}); f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{});
  f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{});
}

// The epilogues that need the stored activation of their tile.
__host__ __device__ constexpr bool res_reads(int epi) { return epi == EPI_DH || epi == EPI_DH_DENSE; }
// Waves of a workgroup.  K = 512 fills the LDS, so one workgroup of eight waves
// runs per CU; below, two workgroups of four, but at K = 256 one of eight where the
// epilogue reads: sharing the token block leaves 96 KB instead of 32 for what it reads.
__host__ __device__ constexpr int res_waves(int epi, int kp) { return kp == 8 || (kp == 4 && res_reads(epi)) ? 8 : 4; }

// KP = K / 64 panels.
template <int EPI, int KP>
__global__ __launch_bounds__(64 * res_waves(EPI, KP), 2) void resident_kernel(const ResArgs g) {
  constexpr int NW = res_waves(EPI, KP);
  constexpr int PANEL = 128 * 128;   // bytes of one 64-wide panel of the token block
  // READS: each wave brings in the stored activation of its tile, 8 blocks of 16
  // tokens (SKB KB each).  The first SLOTS are copied by DMA to LDS of its own at
  // the tile's start (with the codes of all 128 tokens of a compressed S, 1 KB),
  // the next REGS loaded to registers at the epilogue's start, where the fragments'
  // are free (as many as there are without spills), and any left copied to slots that
  // have come free.  An epilogue then waits for about one memory latency, not for one
  // per 3 (dense: 2) blocks.  Microseconds before and after: dense dH at 350M, 32768
  // tokens 131 / 123, at 1B, 16384 tokens 153 / 147; masked dH at 350M, 16381 tokens
  // 42 / 39, at 1B, 65536 tokens 340 / 334.  (Cached instead of streaming reads: dense
  // dH 120, but dP, which finds less of dH in the caches, 63 -> 71.)
  constexpr bool READS = res_reads(EPI);
  constexpr int SKB = EPI == EPI_DH ? 1 : 2, CODES = EPI == EPI_DH ? 1024 : 0;
  constexpr int SLOTS = KP == 8 ? (EPI == EPI_DH ? 3 : 2) : (EPI == EPI_DH ? 8 : 6);
  constexpr int REGS = KP == 8 ? (EPI == EPI_DH ? 3 : 4) : EPI == EPI_DH ? 0 : KP == 4 ? 1 : 2;
  constexpr int AHEAD = SLOTS + REGS;
  constexpr int SBUF = SLOTS * SKB * 1024 + CODES;
  constexpr int LDS = KP * PANEL + (READS ? NW * SBUF : 0);
  __shared__ __attribute__((aligned(1024))) char smem[LDS];
  // Waves take feature blocks from a counter (the two waves of a SIMD share it
  // unevenly, so a fixed deal ends ragged: k2 at 1B 313 against 297 us); where
  // the tile's S fills the LDS to the last byte they are dealt in turn.
  constexpr bool COUNTER = LDS * (8 / NW) < 160 * 1024;
  __shared__ int s_next;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fs = (int)blockIdx.x % g.fsplit;
  const int64_t n0 = (int64_t)((int)blockIdx.x / g.fsplit) * 128;
  const int f_begin = (int)((int64_t)fs * g.nfb / g.fsplit), f_end = (int)((int64_t)(fs + 1) * g.nfb / g.fsplit);
  const int t_end = (int)(g.T - n0 < 128 ? g.T - n0 : 128);   // tokens of this block

  // The token block -> LDS: panel q's row t holds its 8 chunks of 16 bytes, chunk
  // c at position c ^ (t / 2) % 8: the rows and chunks a fragment read serves
  // together (below) then lie in distinct banks.  Rows past the last token are 0.
  const uint32_t smem_lds = lds_u32(smem);
  for (int q = 0; q < KP; ++q) {
#pragma unroll
    for (int k = 0; k < 16 / NW; ++k) {
      const int blk = wave * (16 / NW) + k, row = blk * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
      const void* src = row < t_end ? (const void*)(g.X + (n0 + row) * g.ldx + q * 64 + c * 8) : (const void*)g_dma_zero;
      dma_b128(src, __builtin_amdgcn_readfirstlane(smem_lds + q * PANEL + blk * 1024));
    }
  }
  if constexpr (COUNTER) {
    if (tid == 0) s_next = f_begin + NW;
  }
  // Weights: ring of one K panel (2 k32 steps x 4 row quarters)
  u32x4 a[2][4];
  const u32x4* W = (const u32x4*)g.W;
  auto load_a = [&](const u32x4* p, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[kk][i] = *(const gu32x4*)(p + kk * 256 + i * 64 + lane);
  };
  auto block_ptr = [&](int fb) __attribute__((always_inline)) { return (const u32x4*)uniform_ptr(W + (int64_t)fb * KP * 512); };

  int cur = f_begin + wave;
  const u32x4* wp = block_ptr(cur < f_end ? cur : f_begin);
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) load_a(wp, kk);
  wait_vmcnt<0>();
  __syncthreads();
  if (cur >= f_end) return;

  // Token fragments: row 16 j + l % 16 of a panel, chunk 4 kk + l / 16.
  const int l16 = lane & 15, lg = lane >> 4;
  bf16x8 bf[2][4];
  const char* xb[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) xb[x] = smem + l16 * 128 + ((lg | 4 * x) ^ (l16 >> 1)) * 16;
  // sub-step s of a panel: k32 step s / 2, tokens 64 (s % 2) .. + 63
  auto read_b = [&](int q, int s, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) bf[slot][j] = *(const bf16x8*)(xb[s >> 1] + q * PANEL + (4 * (s & 1) + j) * 2048);
  };
  f32x4 acc[4][8];
  auto panel = [&](auto first, auto last, int q, const u32x4* np) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // (the next tile's first fragments are read after the epilogue)
      if (s < 3 || !decltype(last)::value) read_b(s < 3 ? q : q + 1, (s + 1) & 3, (s + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      const int kk = s >> 1, j0 = 4 * (s & 1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 z = {0.f, 0.f, 0.f, 0.f};
          acc[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[kk][i]), bf[s & 1][j],
                                                                  decltype(first)::value && kk == 0 ? z : acc[i][j0 + j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      if (s & 1) load_a(np, kk);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Dense rows: after a permlane16 swap of the two row quarters of a pair,
  // lane group lg holds 8 consecutive features from 16 (lg % 2) + 8 (lg / 2) of
  // the pair's 32, so a store covers 64 bytes of each of 16 token rows.
  char* sbuf = smem + KP * PANEL + wave * SBUF;   // this wave's stored activation (READS)
  const uint32_t sbuf_lds = lds_u32(sbuf);
  // Copies token block j of feature block fb, lane l's 16 bytes to slot byte
  // 16 l: the piece the epilogue's lane l reads.  (Rows past the last token and
  // features past the last re-read a valid piece; nothing uses them.)
  // (j - AHEAD: the block whose slot a later copy takes)
  auto copy_s = [&](int fb, int j) __attribute__((always_inline)) {
    if constexpr (READS) {
      int le = lane;   // laundered: offsets formed here, not kept live
      asm volatile("" : "+v"(le));
      int row = j * 16 + (le & 15);
      row = row < t_end ? row : 0;
      const uint32_t slot = sbuf_lds + (j < SLOTS ? j : j - AHEAD) * SKB * 1024;
      if constexpr (EPI == EPI_DH) {
        const int64_t tb = n0 & ~(int64_t)255;
        const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
        dma_b128_nt_s(g.sv + tb * g.ldv + (int64_t)fb * R * 32 + (n0 - tb) * 32, (uint32_t)(row * 64 + (le >> 4) * 16), slot);
      } else {
        const int f = 16 * ((le >> 4) & 1) + 8 * (le >> 5), left = g.f_valid - fb * 64;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int fh = f + 32 * h < left ? f + 32 * h : 0;
          dma_b128_nt_s(g.act + n0 * g.ld_act + fb * 64, (uint32_t)row * (uint32_t)(g.ld_act * 2) + fh * 2, slot + h * 1024);
        }
      }
    }
  };
  auto copy_codes = [&](int fb) __attribute__((always_inline)) {
    if constexpr (EPI == EPI_DH) {
      int le = lane;
      asm volatile("" : "+v"(le));
      const int64_t tb = n0 & ~(int64_t)255;
      const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        int row = h * 32 + (le >> 1);
        row = row < t_end ? row : 0;
        dma_b32_nt_s(g.sm + tb * g.ldm + (int64_t)fb * R * 8 + (n0 - tb) * 8, (uint32_t)(row * 8 + (le & 1) * 4),
                     sbuf_lds + SLOTS * SKB * 1024 + h * 256);
      }
    }
  };
  // The REGS blocks after those, the same pieces to registers.
  u32x4 sreg[REGS > 0 ? REGS * SKB : 1];
  auto load_s = [&](int fb, int le) __attribute__((always_inline)) {
    if constexpr (READS) {
#pragma unroll
      for (int k = 0; k < REGS; ++k) {
        int row = (SLOTS + k) * 16 + (le & 15);
        row = row < t_end ? row : 0;
        if constexpr (EPI == EPI_DH) {
          const int64_t tb = n0 & ~(int64_t)255;
          const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
          const char* p = (const char*)uniform_ptr(g.sv + tb * g.ldv + (int64_t)fb * R * 32 + (n0 - tb) * 32);
          sreg[k] = __builtin_nontemporal_load((const gu32x4*)(p + (uint32_t)(row * 64 + (le >> 4) * 16)));
        } else {
          const int f = 16 * ((le >> 4) & 1) + 8 * (le >> 5), left = g.f_valid - fb * 64;
          const char* p = (const char*)uniform_ptr(g.act + n0 * g.ld_act + fb * 64);
#pragma unroll
          for (int h = 0; h < 2; ++h)
            sreg[2 * k + h] = __builtin_nontemporal_load(
                (const gu32x4*)(p + (uint32_t)((uint32_t)row * (uint32_t)(g.ld_act * 2) + (f + 32 * h < left ? f + 32 * h : 0) * 2)));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Waits for the copy of token block j.  The first SLOTS are older than the
  // weight loads of the last panel (8 of them follow).  Later ones follow the
  // stores of block j - AHEAD; after them come AHEAD - 1 blocks' stores and the
  // copies of the blocks below 8 among those.  Where a store may have been
  // skipped (ragged tiles) everything is waited for.
  auto wait_s = [&](auto jc, bool full) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if constexpr (j == 0) {
      wait_vmcnt<8>();
    } else if constexpr (j >= AHEAD) {
      constexpr int copies = 7 - j < AHEAD - 1 ? 7 - j : AHEAD - 1;
      if (full) wait_vmcnt<SKB * (AHEAD - 1 + copies)>();
      else wait_vmcnt<0>();
    }
  };
  for (;;) {
    int nxt = cur + NW;
    if constexpr (COUNTER) {
      if (lane == 0) nxt = atomicAdd(&s_next, 1);
      nxt = __builtin_amdgcn_readfirstlane(nxt);
    }
    if constexpr (READS) {
      copy_codes(cur);
#pragma unroll
      for (int j = 0; j < SLOTS; ++j) copy_s(cur, j);
    }
    read_b(0, 0, 0);
    panel(std::true_type{}, std::false_type{}, 0, wp + 512);
#pragma unroll
    for (int q = 1; q + 1 < KP; ++q) panel(std::false_type{}, std::false_type{}, q, wp + (q + 1) * 512);
    const u32x4* wn = block_ptr(nxt < f_end ? nxt : cur);
    panel(std::false_type{}, std::true_type{}, KP - 1, wn);
    __builtin_amdgcn_s_setprio(1);
    // ---- epilogue: features 64 cur .. + 63.  Element e of acc[i][j] in lane l
    // is feature 16 i + 4 lg + e (lg = l / 16) of token 16 j + l % 16: one whole
    // group of 4.
    // (lane index laundered, so that the store offsets are formed here and
    // not kept live across the main loop)
    int le = lane;
    asm volatile("" : "+v"(le));
    const int e16 = le & 15, eg = le >> 4;
    if constexpr (EPI == EPI_SPARSIFY) {
      const int64_t tb = n0 & ~(int64_t)255;
      const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
      char* dv = (char*)uniform_ptr(g.sv + tb * g.ldv + (int64_t)cur * R * 32 + (n0 - tb) * 32);
      char* dm = (char*)uniform_ptr(g.sm + tb * g.ldm + (int64_t)cur * R * 8 + (n0 - tb) * 8);
#pragma unroll
      for (int jj = 0; jj < 8; jj += 4) {
        uint32_t w[2][4];   // code of group 4 i + lg at bits 16 (i % 2) + 4 lg of word i / 2, per token block
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = jj + u;
          uint32_t v[4], c[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t p01 = bf16x2_rne(relu_f32(acc[i][j][0]), relu_f32(acc[i][j][1]));
            const uint32_t p23 = bf16x2_rne(relu_f32(acc[i][j][2]), relu_f32(acc[i][j][3]));
            const Top2 t = top2_keys_hi(p01, p23);
            c[i] = top2_code_xor15(t);
            const float x = __builtin_bit_cast(float, t.first << 2), y = __builtin_bit_cast(float, t.second << 2);
            v[i] = bf16x2_rne(x * x, y * y);
          }
#pragma unroll
          for (int h = 0; h < 2; ++h) w[h][u] = ((c[2 * h] | (c[2 * h + 1] << 16)) ^ 0x000F000Fu) << (4 * eg);
          transpose4(v);   // lane group lg gets the 16 bytes of row quarter i = lg
          if (j * 16 + e16 < t_end) *(gu32x4*)(dv + j * 1024 + (uint32_t)(e16 * 64 + eg * 16)) = u32x4{v[0], v[1], v[2], v[3]};
          __builtin_amdgcn_sched_barrier(0);
        }
        // each token's word is the OR over its four lane groups
        uint32_t o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const auto s0 = __builtin_amdgcn_permlane32_swap(w[h][0], w[h][2], false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(w[h][1], w[h][3], false, false);
          const auto s2 = __builtin_amdgcn_permlane16_swap(s0[0] | s0[1], s1[0] | s1[1], false, false);
          o[h] = s2[0] | s2[1];
        }
        if (jj * 16 + le < t_end) *(gu32x2*)(dm + jj * 128 + (uint32_t)(le * 8)) = u32x2{o[0], o[1]};
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (EPI == EPI_DH) {
      // dS at the kept positions times 2 relu(h), relu(h) = bf16(sqrt(s)) exactly
      const int64_t tb = n0 & ~(int64_t)255;
      const int64_t R = g.T - tb < 256 ? g.T - tb : 256;
      char* dv = (char*)uniform_ptr(g.dv + tb * g.ldv + (int64_t)cur * R * 32 + (n0 - tb) * 32);
      const char* sl = sbuf + le * 16;
      const char* sc = sbuf + SLOTS * 1024 + e16 * 8;
      wait_s(std::integral_constant<int, 0>{}, true);
      load_s(cur, le);
      unroll8([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j > 0) wait_s(jc, t_end == 128);
        const u32x4 sv = j >= SLOTS && j < AHEAD ? sreg[j >= SLOTS && j < AHEAD ? j - SLOTS : 0]
                                                 : *(const u32x4*)(sl + (j < SLOTS ? j : j - AHEAD) * 1024);
        const u32x2 m = *(const u32x2*)(sc + j * 128);
        uint32_t v[4] = {sv[0], sv[1], sv[2], sv[3]};
        // a subnormal s, which the raw square root flushes (bit pattern v in
        // [1, 0x7F], tested as (v - 1) mod 2^16 < 0x7F on the smallest)
        u16x2 vmin = {0xFFFFu, 0xFFFFu};
#pragma unroll
        for (int i = 0; i < 4; ++i) vmin = __builtin_elementwise_min(vmin, __builtin_bit_cast(u16x2, v[i]) - (u16x2){1u, 1u});
        const bool tiny = (vmin[0] < vmin[1] ? vmin[0] : vmin[1]) < 0x7Fu;
        transpose4(v);
        float rt[4][2];
        if (__builtin_amdgcn_ballot_w64(tiny) == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            rt[i][0] = __builtin_amdgcn_sqrtf(__builtin_bit_cast(float, v[i] << 16));
            rt[i][1] = __builtin_amdgcn_sqrtf(__builtin_bit_cast(float, v[i] & 0xFFFF0000u));
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            rt[i][0] = sqrt_for_bf16(__builtin_bit_cast(float, v[i] << 16));
            rt[i][1] = sqrt_for_bf16(__builtin_bit_cast(float, v[i] & 0xFFFF0000u));
          }
        }
        const uint32_t w0 = m[0] >> (4 * eg), w1 = m[1] >> (4 * eg);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t w = i < 2 ? w0 : w1;
          const uint32_t i0 = __builtin_amdgcn_ubfe(w, 16 * (i & 1), 2), i1 = __builtin_amdgcn_ubfe(w, 16 * (i & 1) + 2, 2);
          const f32x4 ds = acc[i][j];
          const float d0 = i0 == 0u ? ds[0] : i0 == 1u ? ds[1] : ds[2];
          const float d1 = i1 == 1u ? ds[1] : i1 == 2u ? ds[2] : ds[3];
          const uint32_t rr = bf16x2_rne(rt[i][0], rt[i][1]);   // relu(h), exact
          v[i] = bf16x2_rne(d0 * 2.0f * __builtin_bit_cast(float, rr << 16),
                            d1 * 2.0f * __builtin_bit_cast(float, rr & 0xFFFF0000u));
        }
        transpose4(v);
        if (j * 16 + e16 < t_end) *(gu32x4*)(dv + j * 1024 + (uint32_t)(e16 * 64 + eg * 16)) = u32x4{v[0], v[1], v[2], v[3]};
        if constexpr (j + AHEAD < 8) copy_s(cur, j + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    if constexpr (EPI == EPI_BF16 || EPI == EPI_ACT_DENSE || EPI == EPI_DH_DENSE) {
      const int f = cur * 64 + 16 * (eg & 1) + 8 * (eg >> 1);
      if constexpr (READS) {
        wait_s(std::integral_constant<int, 0>{}, true);
        load_s(cur, le);
      }
      unroll8([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        uint16_t* dst = g.C + (n0 + j * 16 + e16) * g.ldc + f;
        const bool ok = j * 16 + e16 < t_end;
        u32x4 sin[2];
        if constexpr (EPI == EPI_DH_DENSE) {
          if constexpr (j > 0) wait_s(jc, t_end == 128 && cur * 64 + 64 <= g.f_valid);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if constexpr (j >= SLOTS && j < AHEAD) sin[h] = sreg[2 * (j - SLOTS) + h];
            else sin[h] = *(const u32x4*)(sbuf + ((j < SLOTS ? j : j - AHEAD) * 2 + h) * 1024 + le * 16);
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t m[2][2];   // row quarter 2h + p, feature pair e
          if constexpr (EPI == EPI_DH_DENSE) {
            // the stored s in the accumulators' places, its exact root relu(h)
            u16x2 vmin = {0xFFFFu, 0xFFFFu};
#pragma unroll
            for (int e = 0; e < 4; ++e) vmin = __builtin_elementwise_min(vmin, __builtin_bit_cast(u16x2, (uint32_t)sin[h][e]) - (u16x2){1u, 1u});
            const bool tiny = (vmin[0] < vmin[1] ? vmin[0] : vmin[1]) < 0x7Fu;
            uint32_t q[2][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const auto sw = __builtin_amdgcn_permlane16_swap(sin[h][e], sin[h][2 + e], false, false);
              q[0][e] = sw[0];
              q[1][e] = sw[1];
            }
            const bool any_tiny = __builtin_amdgcn_ballot_w64(tiny) != 0;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                const float s0 = __builtin_bit_cast(float, q[p][e] << 16), s1 = __builtin_bit_cast(float, q[p][e] & 0xFFFF0000u);
                float r0, r1;
                if (!any_tiny) {
                  r0 = __builtin_amdgcn_sqrtf(s0);
                  r1 = __builtin_amdgcn_sqrtf(s1);
                } else {
                  r0 = sqrt_for_bf16(s0);
                  r1 = sqrt_for_bf16(s1);
                }
                const uint32_t rr = bf16x2_rne(r0, r1);
                m[p][e] = bf16x2_rne(acc[2 * h + p][j][2 * e] * 2.0f * __builtin_bit_cast(float, rr << 16),
                                     acc[2 * h + p][j][2 * e + 1] * 2.0f * __builtin_bit_cast(float, rr & 0xFFFF0000u));
              }
          } else {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                const float x = acc[2 * h + p][j][2 * e], y = acc[2 * h + p][j][2 * e + 1];
                if constexpr (EPI == EPI_ACT_DENSE) {
                  // h relu'd and rounded to bf16, squared and rounded
                  const uint32_t r = bf16x2_rne(relu_f32(x), relu_f32(y));
                  const float lo = __builtin_bit_cast(float, r << 16), hi = __builtin_bit_cast(float, r & 0xFFFF0000u);
                  m[p][e] = bf16x2_rne(lo * lo, hi * hi);
                } else {
                  m[p][e] = bf16x2_rne(x, y);
                }
              }
          }
          const auto x = __builtin_amdgcn_permlane16_swap(m[0][0], m[1][0], false, false);
          const auto y = __builtin_amdgcn_permlane16_swap(m[0][1], m[1][1], false, false);
          if (ok && f + 32 * h < g.f_valid) *(u32x4*)(dst + 32 * h) = u32x4{x[0], y[0], x[1], y[1]};
        }
        if constexpr (READS && j + AHEAD < 8) copy_s(cur, j + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    __builtin_amdgcn_s_setprio(0);
    if (nxt >= f_end) break;
    cur = nxt;
    wp = wn;
  }
}

}  // namespace elas
