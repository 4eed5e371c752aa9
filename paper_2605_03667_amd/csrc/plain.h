// Tiled dense product with a plain output for gfx950: C [M x N] = A B^T in bf16
// (or fp32 split-K partials), A [M x K], B [N x K] or blocked.
//
// A persistent workgroup per CU (two for the 128 x 128 tiles) walks its tiles; each
// wave owns a TM x TN part of the tile.  Both operands go to LDS by DMA, 64 K per
// step, in rings of stages.  The barrier of a step sits before its last MFMA
// sub-step, when the step's fragments are all in registers: the next step's first
// fragment reads run under those MFMAs, and the step's own stage is free for copies
// a whole ring ahead.  Copies run on into the workgroup's next tile.  Rows past the
// end of an operand re-read its last row (their results are not stored), so that
// only a K that is no multiple of 64 takes checked copies.
//
// Bound by the copies' issue (64 KB per step go through the CU's one address unit,
// about half of the step's MFMA time, and hold the waves that issue them) and by
// the barrier; the 16x16x32 MFMA leaves more of the power budget to the clock.
// Measured against the earlier loop (barrier before the first reads, 32x32x16, one
// workgroup per CU, checked copies on ragged tiles; microseconds): 350M shapes, k1 at
// 16381 tokens 25.5 -> 18.5, at 33333 54 -> 35; dense Z at 32768 tokens 88 -> 70, dP
// 80 -> 58; 130M full-rank down product at 8192 tokens 44 -> 33; 1B at 65536 tokens
// 127 -> 130, within what the rest of the step gains from the power left.  Full-rank
// up products with their ReLU^2, which that loop computed transposed, against this
// (with the timing events' few): 60M at 700 tokens 16 -> 13, 350M at 4099 48 -> 33,
// 1B at 2048 79 -> 56 and at 16384 394 -> 351.
#pragma once

#include "gemm.h"

namespace elas {

// SA, SB: stages of A's and of B's ring.
// EPI: EPI_BF16, EPI_F32 (split-K partials) or EPI_ACT_DENSE (relu(.)^2 in bf16).
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int EPI_, int SA_, int SB_>
struct PlainCfg {
  static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, SA = SA_, SB = SB_;
  static constexpr int EPI = EPI_;
  static constexpr int NW = WAVES_M_ * WAVES_N_, NT = 64 * NW, BK = 64;
  static constexpr int TM = BM_ / WAVES_M_, TN = BN_ / WAVES_N_;
  static constexpr int AB = BM_ * 128, BB = BN_ * 128;   // bytes of a stage
  static constexpr int LDS = SA_ * AB + SB_ * BB;
  static_assert(LDS <= 160 * 1024 && SA_ >= SB_ && SA_ <= SB_ + 1 && SB_ >= 2, "rings");
};

template <class Cfg>
__global__ __launch_bounds__(Cfg::NT, 2) void plain_kernel(const GemmArgs g) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, NW = Cfg::NW, TM = Cfg::TM, TN = Cfg::TN, SA = Cfg::SA, SB = Cfg::SB;
  __shared__ __attribute__((aligned(1024))) char smem[Cfg::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / Cfg::WAVES_N, wn = wave % Cfg::WAVES_N;
  const int l16 = lane & 15, lg = lane >> 4;
  // Split-K grids (a multiple of 8 splits): each XCD runs whole splits, whose
  // tiles read the same rows of both operands through its L2.
  int bx = blockIdx.x, by = blockIdx.y;
  if (gridDim.y > 1 && gridDim.y % 8 == 0) {
    const int L = blockIdx.x + gridDim.x * blockIdx.y, x = L % 8, j = L / 8;
    by = x * (gridDim.y / 8) + j / gridDim.x;
    bx = j % gridDim.x;
  }
  const int64_t kbeg = (int64_t)by * g.k_split;
  const int64_t kend = kbeg + g.k_split < g.K ? kbeg + g.k_split : g.K;
  const int nsteps = kend > kbeg ? (int)((kend - kbeg + 63) / 64) : 0;
  const TileRange tr = tile_range(bx, gridDim.x, g.tiles_m * g.tiles_n);
  if (tr.first >= tr.end) return;
  const bool bblk = g.b_nsk > 0;

  // ---- copies: an iterator over the (tile, step) sequence of this workgroup ----
  using DA = DmaTile<BM, 128, false, NW, true>;
  using DB = DmaTile<BN, 128, false, NW, true>;
  constexpr int LA = DA::PER_WAVE, LB = DB::PER_WAVE;
  const uint32_t lds0 = lds_u32(smem);
  uint32_t offA[LA], offB[LB];   // of the tile being copied: rows past the end are the last one
  // Each operand's position: next step of tile `tile` (>= tr.end: none left), its
  // origin, and the unchecked steps (a prefix of a tile's) with their source.
  struct Pos {
    int tile, step, fast;
    int64_t org;
    const char* p;
  };
  auto whole_steps = [&](int64_t k_valid) __attribute__((always_inline)) {
    const int64_t k_in = k_valid - kbeg;
    return __builtin_amdgcn_readfirstlane(k_in <= 0 ? 0 : (int)(k_in / 64 < nsteps ? k_in / 64 : nsteps));
  };
  auto start_a = [&](Pos& c) __attribute__((always_inline)) {
    c.step = 0;
    if (c.tile >= tr.end) return;
    c.org = (int64_t)(c.tile / g.tiles_n) * BM;
    c.fast = whole_steps(g.ka_valid);
    c.p = (const char*)uniform_ptr(DA::step_base(g.A, g.lda, c.org, kbeg));
#pragma unroll
    for (int j = 0; j < LA; ++j) offA[j] = DA::lane_off(j, g.lda, wave, lane, (int)(g.m_valid - c.org < BM ? g.m_valid - c.org : BM));
  };
  auto start_b = [&](Pos& c) __attribute__((always_inline)) {
    c.step = 0;
    if (c.tile >= tr.end) return;
    c.org = (int64_t)(c.tile % g.tiles_n) * BN;
    c.fast = bblk ? nsteps : whole_steps(g.kb_valid);
    c.p = (const char*)uniform_ptr(bblk ? (const char*)(g.B + blocked_index(c.org, kbeg, g.b_nsk)) : DB::step_base(g.B, g.ldb, c.org, kbeg));
    // (the blocked layout is padded to whole panels)
#pragma unroll
    for (int j = 0; j < LB; ++j)
      offB[j] = DB::lane_off(j, bblk ? 64 : g.ldb, wave, lane, bblk || g.N - c.org >= BN ? BN : (int)(g.N - c.org));
  };
  Pos pa{tr.first}, pb{tr.first};
  start_a(pa);
  start_b(pb);
  // Issue the next step's copies into the stage at LDS byte offset `at`.
  auto copy_a = [&](uint32_t at) __attribute__((always_inline)) {
    if (pa.tile >= tr.end) return;
    const uint32_t to = lds0 + at;
    if (pa.step < pa.fast) {
      DA::template issue_fast<0, LA>(pa.p, offA, to, wave);
      pa.p += 128;
    } else {
      int64_t kc = uniform_i64(kbeg + (int64_t)pa.step * 64);
      int lc = lane;   // laundered: addresses formed here, not kept across the loop
      asm volatile("" : "+s"(kc), "+v"(lc));
      DA::template issue<0, LA>(g.A, g.lda, pa.org, g.m_valid, kc, g.ka_valid, to, wave, lc);
    }
    if (++pa.step >= nsteps) {
      pa.tile += tr.stride;
      start_a(pa);
    }
  };
  auto copy_b = [&](uint32_t at) __attribute__((always_inline)) {
    if (pb.tile >= tr.end) return;
    const uint32_t to = lds0 + SA * Cfg::AB + at;
    if (pb.step < pb.fast) {
      DB::template issue_fast<0, LB>(pb.p, offB, to, wave);
      pb.p += bblk ? 32768 : 128;
    } else {
      int64_t kc = uniform_i64(kbeg + (int64_t)pb.step * 64);
      int lc = lane;
      asm volatile("" : "+s"(kc), "+v"(lc));
      DB::template issue<0, LB>(g.B, g.ldb, pb.org, g.N, kc, g.kb_valid, to, wave, lc);
    }
    if (++pb.step >= nsteps) {
      pb.tile += tr.stride;
      start_b(pb);
    }
  };

  // ---- fragments and MFMAs of one step, in four sub-steps ----
  // Sub-step q: k32 step q / 2 against half q % 2 of B's 16-column blocks; the MFMAs
  // take B first, so that a lane accumulates consecutive columns.
  constexpr int FM = TM / 16, FN = TN / 16, NH = FN / 2;
  f32x4 acc[FM][FN];
  bf16x8 af[2][FM], bf[2][NH];
  auto read = [&](const char* sA, const char* sB, int q) __attribute__((always_inline)) {
    const int kk = q >> 1;
    if ((q & 1) == 0) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = wm * TM + i * 16 + l16;
        af[kk][i] = *(const bf16x8*)(sA + row * 128 + swz_pair(row, 4 * kk + lg) * 16);
      }
    }
#pragma unroll
    for (int j = 0; j < NH; ++j) {
      const int row = wn * TN + ((q & 1) * NH + j) * 16 + l16;
      bf[q & 1][j] = *(const bf16x8*)(sB + row * 128 + swz_pair(row, 4 * kk + lg) * 16);
    }
  };
  auto mfma = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NH; ++j)
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        f32x4& c = acc[i][(q & 1) * NH + j];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[q & 1][j], af[q >> 1][i], c, 0, 0, 0);
      }
  };

  // ---- the step sequence ----
  // Stage of the g-th step: g % SA, g % SB.  Before step 0 the copies of SA (SB)
  // steps are issued; at the barrier of step s those of step s + SB of B, then of
  // step s + SA of A, into the stages step s has just left.
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    copy_b(s * Cfg::BB);
    copy_a(s * Cfg::AB);
  }
  if constexpr (SA > SB) copy_a(SB * Cfg::AB);
  const int64_t total = (int64_t)nsteps * ((tr.end - tr.first + tr.stride - 1) / tr.stride);   // steps of all tiles
  int64_t left = total;   // steps not yet finished, the current one included
  int ra = 0, rb = 0;     // stages of the current step
  for (int tile = tr.first; tile < tr.end; tile += tr.stride) {
    const int64_t m0 = (int64_t)(tile / g.tiles_n) * BM, n0 = (int64_t)(tile % g.tiles_n) * BN;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (nsteps > 0) {
      // (a later tile's first step has landed at the previous tile's last barrier)
      if (tile == tr.first) {
        wait_vmcnt<0>();
        lds_barrier();
      }
      read(smem + ra * Cfg::AB, smem + SA * Cfg::AB + rb * Cfg::BB, 0);
    }
    for (int s = 0; s < nsteps; ++s) {
      const char *sA = smem + ra * Cfg::AB, *sB = smem + SA * Cfg::AB + rb * Cfg::BB;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        read(sA, sB, q + 1);
        __builtin_amdgcn_sched_barrier(0);
        mfma(q);
        __builtin_amdgcn_sched_barrier(0);
      }
      const uint32_t fa = ra * Cfg::AB, fb = rb * Cfg::BB;
      ra = ra + 1 == SA ? 0 : ra + 1;
      rb = rb + 1 == SB ? 0 : rb + 1;
      // Step s + 1's copies have landed once only those issued after them are in
      // flight: A's of step s + 2 (after B's of s + 1) and, with SB > 2, both of the
      // steps up to s + SB - 1.
      if (left > SA) {
        wait_vmcnt<(SA > SB ? LA : 0) + (SB - 2) * (LA + LB)>();
      } else {
        wait_vmcnt<0>();
      }
      lds_wait_barrier();   // every wave's copies; this step's fragments are in registers
      if (s + 1 < nsteps) read(smem + ra * Cfg::AB, smem + SA * Cfg::AB + rb * Cfg::BB, 0);
      __builtin_amdgcn_sched_barrier(0);
      mfma(3);
      __builtin_amdgcn_sched_barrier(0);
      copy_b(fb);
      copy_a(fa);
      --left;
    }
    // ---- epilogue ----
    // element e of acc[i][j] in lane l is C[row l % 16][col 4 (l / 16) + e] of its
    // block; N is a multiple of 8
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int64_t row = m0 + wm * TM + i * 16 + l16;
      if constexpr (Cfg::EPI != EPI_F32) {
        auto out = [&](float x, float y) __attribute__((always_inline)) {
          if constexpr (Cfg::EPI == EPI_ACT_DENSE) {
            // h relu'd and rounded to bf16, squared and rounded
            const uint32_t r = bf16x2_rne(relu_f32(x), relu_f32(y));
            const float lo = __builtin_bit_cast(float, r << 16), hi = __builtin_bit_cast(float, r & 0xFFFF0000u);
            return bf16x2_rne(lo * lo, hi * hi);
          } else {
            return bf16x2_rne(x, y);
          }
        };
        // after a permlane16 swap of two neighbouring blocks lane group lg holds 8
        // consecutive columns from 16 (lg % 2) + 8 (lg / 2) of their 32
#pragma unroll
        for (int j = 0; j < FN; j += 2) {
          const int64_t col = n0 + wn * TN + j * 16 + 16 * (lg & 1) + 8 * (lg >> 1);
          const auto x = __builtin_amdgcn_permlane16_swap(out(acc[i][j][0], acc[i][j][1]),
                                                          out(acc[i][j + 1][0], acc[i][j + 1][1]), false, false);
          const auto y = __builtin_amdgcn_permlane16_swap(out(acc[i][j][2], acc[i][j][3]),
                                                          out(acc[i][j + 1][2], acc[i][j + 1][3]), false, false);
          if (row < g.M && col < g.N) *(uint4*)((__bf16*)g.C + row * g.ldc + col) = make_uint4(x[0], y[0], x[1], y[1]);
        }
      } else {
        float* part = (float*)g.C + (int64_t)by * g.M * g.N;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int64_t col = n0 + wn * TN + j * 16 + 4 * lg;
          if (row < g.M && col < g.N) *(f32x4*)(part + row * g.N + col) = acc[i][j];
        }
      }
    }
  }
}

}  // namespace elas
