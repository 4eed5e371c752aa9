// Weight gradients of one backward in one launch, for gfx950: every product
// C = A^T B over the T tokens (dV_down = Z^T dY, dU_down = S^T dZ, dV_up^T = dH^T P,
// dU_up = x^T dP).  All contract over the same tokens, so their output tiles form
// one list, and the tokens are cut into as few chunks as fill the chip with one
// (tile, chunk) unit per workgroup.  Launched one by one, a product of 4 tiles
// needed 64 splits to fill the chip, and wrote and read 64 fp32 partials of its
// output.  The partials are added in chunk (= K) order by one reduce launch, so
// results are deterministic.  Neighbouring units, the tiles of one chunk, run on
// one XCD at the same time and share the operands' rows in its L2; equal shares of
// the whole (tile, step) list (stream-K) fill the chip a little better but share
// nothing, and read three times as much.
// Measured against one launch and one reduce per product (microseconds, with the
// reduces): 60M at 2048 tokens 119 -> 22, 130M at 8192 119 -> 51, 350M at 16384
// 192 -> 95 and at 65536 395 -> 291, 1B at 65536 1099 -> 1071.
//
// A tile is 256 x 256 on 8 waves or, where that leaves shares of a few steps,
// 128 x 128 on 4.  Operands are token-major: dense ones go to LDS as stored, by
// DMA, and are read with the transposing ds_read_b64_tr_b16; the compressed one
// (S or dH, 2:4 along features) is expanded in registers on the way.  The barrier
// of a step sits before its last MFMA sub-step, whose fragments are in registers
// by then, so that the next step's first reads and copies run under MFMAs.
// The compressed products take about 4000 cycles per step for 2048 of MFMAs: the
// copies' issue and landing, the expansion and the barrier (stamped: 1000, 350,
// 400 and 900) do not overlap them all; the chip is far from its memory rates.
#pragma once

#include "gemm.h"

namespace elas {

// ---- K-major tiles ----------------------------------------------------------
// LDS row k (one per token of the step, 64 of them) holds the tile's ROWS
// elements, in 32-byte chunks of 16 elements; chunk c of row k sits at chunk
// position c ^ 2 (k & 3) ^ (k / 8) % 2.
//
// ds_read_b64_tr_b16 (gfx950, pinned by a probe): within each group of 16
// lanes, lane j reads 4 consecutive 16-bit elements; lane i of the group then
// receives element i % 4 of lane 4q + i/4's read, for q = 0..3.  When lane j
// reads row k0 + j/4 at columns c0 + 4 (j % 4), lane i therefore receives
// column c0 + i of rows k0..k0+3: one MFMA fragment half.  The 32 lanes
// served together touch rows k0..k0+3 and k0+8..k0+11 at one logical chunk; the
// swizzle spreads these eight 32-byte pieces over eight distinct positions,
// i.e. all 64 banks (each row is a multiple of 256 bytes).
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int km_swz(int k, int chunk) { return chunk ^ ((k & 3) << 1) ^ ((k >> 3) & 1); }

// Fragment of a v_mfma_f32_16x16x32_bf16 operand from a K-major LDS tile:
// lane l gets column col0 + l % 16 (col0 a multiple of 16), contraction indices
// 32 kk + 8 (l / 16) + 0..7.  km_lane is the lane's address for kk = 0, from
// which the fragment's two halves and kk lie at constant offsets.
template <int ROWS>
__device__ __forceinline__ const char* km_lane(const char* base, int col0, int lane) {
  const int j = lane & 15, k = 8 * (lane >> 4) + (j >> 2);
  return base + k * (ROWS * 2) + (km_swz(k, col0 >> 4) << 5) + (j & 3) * 8;
}
template <int ROWS>
__device__ __forceinline__ bf16x8 frag_km(const char* p) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * ROWS * 2));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// A dense K-major tile [64 x ROWS] copied by DMA: 1 KB blocks, PER_WAVE per
// wave; lane i fills the block's 16-byte unit i, i.e. physical unit (i mod
// units per row) of row (block rows + i / units per row), and fetches the
// global 8 elements that the swizzle maps there.
template <int ROWS, int NW>
struct DmaTileKM {
  static constexpr int ROWB = ROWS * 2;
  static constexpr int BLOCKS = 64 * ROWB / 1024;
  static constexpr int PER_WAVE = BLOCKS / NW;
  static_assert(BLOCKS % NW == 0 && ROWB <= 1024, "blocks per wave");
  template <int J0, int J1>
  __device__ __forceinline__ static void issue(const uint16_t* __restrict__ p, int64_t ld, int64_t col0,
                                               int64_t cols_valid, int64_t k0, int64_t k_valid, uint32_t lds,
                                               int wave, int lane) {
#pragma unroll
    for (int j = J0; j < J1; ++j) {
      const int blk = wave * PER_WAVE + j;
      const int off = blk * 1024 + lane * 16;
      const int k = off / ROWB, pu = (off % ROWB) / 16;
      const int col = km_swz(k, pu >> 1) * 16 + (pu & 1) * 8;
      const int64_t gk = k0 + k, gc = col0 + col;
      const void* src = (gk < k_valid && gc < cols_valid) ? (const void*)(p + gk * ld + gc) : (const void*)g_dma_zero;
      dma_b128(src, __builtin_amdgcn_readfirstlane(lds + blk * 1024));
    }
  }
  __device__ __forceinline__ static uint32_t lane_off(int j, int64_t ld, int wave, int lane) {
    const int blk = wave * PER_WAVE + j;
    const int off = blk * 1024 + lane * 16;
    const int k = off / ROWB, pu = (off % ROWB) / 16;
    const int col = km_swz(k, pu >> 1) * 16 + (pu & 1) * 8;
    return (uint32_t)k * (uint32_t)(ld * 2) + (uint32_t)col * 2u;
  }
  __device__ __forceinline__ static const char* step_base(const uint16_t* p, int64_t ld, int64_t col0, int64_t k0) {
    return (const char*)(p + k0 * ld + col0);
  }
  template <int J0, int J1>
  __device__ __forceinline__ static void issue_fast(const char* sbase, const uint32_t* voff, uint32_t lds, int wave, int from = J0, int to = J1) {
#pragma unroll
    for (int j = J0; j < J1; ++j)
      if (j >= from && j < to) dma_b128_s(sbase, voff[j], lds + (wave * PER_WAVE + j) * 1024);
  }
};

// A 2:4 K-major tile: rows of kept values [K x cols/2] + metadata [K x cols/8]
// (the compressed activation read along tokens).  Each thread loads the kept
// values (16 bytes) and codes (2 bytes) of 16 consecutive features of one
// contraction row, and after the current step's MFMAs writes them expanded
// (32 bytes) into the K-major LDS tile; no transpose is needed.
template <int ROWS, int NT>
struct StagerKMSP {
  static constexpr int ROWB = ROWS * 2;
  static constexpr int CHUNKS = ROWS / 16;
  static constexpr int NU = 64 * CHUNKS / NT;
  static_assert((64 * CHUNKS) % NT == 0, "units per thread");
  // Unit q (16 features of one contraction row): chunk q % 4 of entry block
  // q / 256 (64 features) at row (q / 4) % 64, so that the 64 lanes of a wave
  // read 16 rows x 64 bytes of one entry block, 1 KB contiguous in the tiled
  // layout.
  __device__ __forceinline__ static int unit_k(int q) { return (q >> 2) & 63; }
  __device__ __forceinline__ static int unit_c(int q) { return (q >> 8) * 4 + (q & 3); }
  uint4 v[NU];
  uint16_t m[NU];
  // The compressed tensor is in the tiled layout with tok rows (tokens =
  // contraction rows here).
  // The step's rows k0 .. k0+63 lie in one block of 256 rows (R of them
  // exist), so every piece is a 32-bit offset from the step's block start.
  __device__ __forceinline__ void load(const uint16_t* __restrict__ pv, int64_t ldv, const uint8_t* __restrict__ pm,
                                       int64_t ldm, int64_t col0, int64_t cols_valid, int64_t k0, int64_t k_valid,
                                       int tid, int64_t tok) {
    const int64_t tb0 = k0 & ~(int64_t)255;
    const int R = (int)(tok - tb0 < 256 ? tok - tb0 : 256);
    const uint16_t* vb = pv + tiled_step<32>(k0, col0, tok, ldv);
    const uint8_t* mb = pm + tiled_step<8>(k0, col0, tok, ldm);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int q = u * NT + tid, k = unit_k(q), c = unit_c(q);
      const int64_t gk = k0 + k, f = col0 + 16 * c;
      v[u] = make_uint4(0u, 0u, 0u, 0u);
      m[u] = 0u;
      if (gk < k_valid && f < cols_valid) {
        v[u] = *(const uint4*)(vb + ((c >> 2) * R * 32 + k * 32 + (c & 3) * 8));
        m[u] = *(const uint16_t*)(mb + ((c >> 2) * R * 8 + k * 8 + (c & 3) * 2));
      }
    }
  }
  // Unchecked path (tile and step inside the matrix, step inside a full block
  // of 256 rows): per-lane byte offsets from the step's block start
  // (tiled_step of its first row and the tile's first column), constant over
  // the steps, and a wave-uniform base per step.  Thread unit (k, c) reads
  // entry block c / 4 at row k, entries 8 (c % 4) .. (values) and 2 (c % 4) ..
  // (metadata bytes).
  __device__ __forceinline__ static void lane_offs(int tid, uint32_t (&ov)[NU], uint32_t (&om)[NU]) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int q = u * NT + tid, k = unit_k(q), c = unit_c(q);
      ov[u] = (uint32_t)((c >> 2) * 256 * 32 + k * 32 + (c & 3) * 8) * 2u;
      om[u] = (uint32_t)((c >> 2) * 256 * 8 + k * 8 + (c & 3) * 2);
    }
  }
  __device__ __forceinline__ void load_fast(const char* vbase, const char* mbase, const uint32_t (&ov)[NU],
                                            const uint32_t (&om)[NU]) {
    const char* vb = (const char*)uniform_ptr(vbase);
    const char* mb = (const char*)uniform_ptr(mbase);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const u32x4 x = *(const __attribute__((address_space(1))) u32x4*)(vb + ov[u]);
      v[u] = make_uint4(x[0], x[1], x[2], x[3]);
      m[u] = *(const __attribute__((address_space(1))) uint16_t*)(mb + om[u]);
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int q = u * NT + tid, k = unit_k(q), c = unit_c(q);
      char* dst = lds + k * ROWB + (km_swz(k, c) << 5);
      *(uint4*)dst = expand2(make_uint2(v[u].x, v[u].y), m[u] & 0xFFu);
      *(uint4*)(dst + 16) = expand2(make_uint2(v[u].z, v[u].w), m[u] >> 8);
    }
  }
};

// One product: A is [T x M] dense, or the compressed S or dH (sparse; tiled, kept
// values with pitch lda and metadata), B [T x N] dense.  Its partial tiles are
// summed into out[m][n], or out[n][m] when transposing, for rows m < rows_out.
struct WgradJob {
  const uint16_t* A;
  int64_t lda;
  const uint8_t* Am;
  int64_t ldam;
  const uint16_t* B;
  int64_t ldb, M, N;
  int sparse, tiles_n, tile0;   // tile0: its first tile in the common list
  float* out;
  int64_t rows_out, ldo;
  int transpose, rblock0, rblocks_n;   // reduce: first 64 x 64 block, blocks along n
};
constexpr int kWgradJobs = 4;
struct WgradArgs {
  WgradJob job[kWgradJobs];
  int64_t T;
  int steps;     // 64-token steps per tile
  int ntiles;    // tiles of all jobs
  int chunks;    // chunks of the steps
  float* part;   // [chunks][ntiles][TB x TB]
};

template <int TB>
__global__ __launch_bounds__(TB == 256 ? 512 : 256, 2) void wgrad_kernel(const WgradArgs g) {
  constexpr int NW = TB == 256 ? 8 : 4, NT = 64 * NW, WAVES_N = 2;
  constexpr int TM = 64, TN = TB / WAVES_N, FM = 4, FN = TN / 16, NH = FN / 2;
  constexpr int OPB = TB * 128;   // bytes of one operand's step
  // A's two stages, then B's: both stages of an operand lie within a read's
  // 16-bit offset, so the loop (unrolled over them) forms no addresses.
  __shared__ __attribute__((aligned(1024))) char smem[4 * OPB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const uint32_t smem_lds = lds_u32(smem);
  using TD = DmaTileKM<TB, NW>;
  using SA = StagerKMSP<TB, NT>;

  f32x4 acc[FM][FN];
  // Accumulates steps [s0, s0 + ns) of the tile at (m0, n0) of job jb.
  auto run = [&](auto sparse, const WgradJob& jb, int64_t m0, int64_t n0, int s0, int ns) __attribute__((always_inline)) {
    constexpr bool SP = decltype(sparse)::value;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t kb = (int64_t)s0 * 64;
    // Steps whose copies need no bounds checks (inside the matrix; the
    // compressed operand's also inside full blocks of 256 tokens), a prefix.
    auto inside = [&](bool tile_in, int64_t k_valid) __attribute__((always_inline)) {
      const int64_t k_in = k_valid - kb;
      return __builtin_amdgcn_readfirstlane(!tile_in || k_in <= 0 ? 0 : (int)(k_in / 64 < ns ? k_in / 64 : ns));
    };
    const int b_in = inside(n0 + TB <= jb.N, g.T);
    const int a_in = inside(m0 + TB <= jb.M, SP ? g.T & ~(int64_t)255 : g.T);
    SA sa;
    uint32_t offA[TD::PER_WAVE], offB[TD::PER_WAVE];
#pragma unroll
    for (int j = 0; j < TD::PER_WAVE; ++j) {
      offB[j] = TD::lane_off(j, jb.ldb, wave, lane);
      offA[j] = SP ? 0 : TD::lane_off(j, jb.lda, wave, lane);
    }
    // Copy cursors (wave-uniform) of the unchecked steps.  In the tiled layout a
    // step's 64 token rows of kept values (metadata) lie 4096 (512) bytes after
    // the previous step's inside a 256-row block; at a block boundary the next
    // block's rows follow 512 lda - 3 * 4096 (256 ldam - 3 * 512) bytes on.
    const char* cb = (const char*)uniform_ptr(TD::step_base(jb.B, jb.ldb, n0, kb));
    const int64_t sb = uniform_i64(jb.ldb * 128);
    const char *cv, *cm = nullptr;
    int64_t jv = 0, jm = 0;
    uint32_t tpos = 0;
    if constexpr (SP) {
      cv = (const char*)uniform_ptr(jb.A + tiled_step<32>(kb, m0, g.T, jb.lda));
      cm = (const char*)uniform_ptr(jb.Am + tiled_step<8>(kb, m0, g.T, jb.ldam));
      jv = uniform_i64(512 * jb.lda - 3 * 4096);
      jm = uniform_i64(256 * jb.ldam - 3 * 512);
      tpos = __builtin_amdgcn_readfirstlane((uint32_t)(kb & 255));
    } else {
      cv = (const char*)uniform_ptr(TD::step_base(jb.A, jb.lda, m0, kb));
      jv = uniform_i64(jb.lda * 128);
    }
    auto stage_lds = [&](int s) __attribute__((always_inline)) { return smem_lds + (uint32_t)((s & 1) * OPB); };
    auto load_a = [&](int s) __attribute__((always_inline)) {
      if constexpr (SP) {
        int tc = tid;   // laundered: offsets formed here, not kept across the loop
        if (s < a_in) {
          asm volatile("" : "+v"(tc));
          uint32_t ov[SA::NU], om[SA::NU];
          SA::lane_offs(tc, ov, om);
          sa.load_fast(cv, cm, ov, om);
          tpos = (tpos + 64) & 255;
          cv += tpos == 0 ? jv : 4096;
          cm += tpos == 0 ? jm : 512;
        } else {
          int64_t kc = uniform_i64(kb + (int64_t)s * 64);
          asm volatile("" : "+s"(kc), "+v"(tc));
          sa.load(jb.A, jb.lda, jb.Am, jb.ldam, m0, jb.M, kc, g.T, tc, g.T);
        }
      } else if (s < a_in) {
        TD::template issue_fast<0, TD::PER_WAVE>(cv, offA, stage_lds(s), wave);
        cv += jv;
      } else {
        TD::template issue<0, TD::PER_WAVE>(jb.A, jb.lda, m0, jb.M, kb + (int64_t)s * 64, g.T, stage_lds(s), wave, lane);
      }
    };
    auto load_b = [&](int s) __attribute__((always_inline)) {
      if (s < b_in) {
        TD::template issue_fast<0, TD::PER_WAVE>(cb, offB, stage_lds(s) + 2 * OPB, wave);
        cb += sb;
      } else {
        TD::template issue<0, TD::PER_WAVE>(jb.B, jb.ldb, n0, jb.N, kb + (int64_t)s * 64, g.T, stage_lds(s) + 2 * OPB, wave, lane);
      }
    };
    auto store_a = [&](int s) __attribute__((always_inline)) {
      if constexpr (SP) sa.store(smem + (s & 1) * OPB, tid);
    };
    const char *pa[FM], *pb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) pa[i] = km_lane<TB>(smem, wm * TM + i * 16, lane);
#pragma unroll
    for (int j = 0; j < FN; ++j) pb[j] = km_lane<TB>(smem + 2 * OPB, wn * TN + j * 16, lane);
    // Sub-step q of a step: k32 step q / 2 against half q % 2 of B's columns.
    bf16x8 af[2][FM], bf[2][NH];
    auto read = [&](int par, int q) __attribute__((always_inline)) {   // par: the stage
      const int off = par * OPB + (q >> 1) * 32 * TB * 2;
      if ((q & 1) == 0) {
#pragma unroll
        for (int i = 0; i < FM; ++i) af[q >> 1][i] = frag_km<TB>(pa[i] + off);
      }
#pragma unroll
      for (int j = 0; j < NH; ++j) bf[q & 1][j] = frag_km<TB>(pb[(q & 1) * NH + j] + off);
    };
    // (hook(j) runs after the MFMAs of column block j)
    auto mfma = [&](int q, auto&& hook) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NH; ++j) {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          f32x4& c = acc[i][(q & 1) * NH + j];
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[q & 1][j], af[q >> 1][i], c, 0, 0, 0);
        }
        hook(j);
      }
    };
    auto nothing = [](int) __attribute__((always_inline)) {};
    load_a(0);
    load_b(0);
    store_a(0);
    if (ns > 1) {
      load_a(1);
      load_b(1);
    }
    if (!SP && ns > 1) wait_vmcnt<2 * TD::PER_WAVE>();
    else wait_vmcnt<0>();
    lds_wait_barrier();
    read(0, 0);
    auto step = [&](auto parity, int s) __attribute__((always_inline)) {
      constexpr int P = decltype(parity)::value;   // s % 2
      read(P, 1);
      __builtin_amdgcn_sched_barrier(0);
      mfma(0, nothing);
      __builtin_amdgcn_sched_barrier(0);
      read(P, 2);
      __builtin_amdgcn_sched_barrier(0);
      mfma(1, nothing);
      __builtin_amdgcn_sched_barrier(0);
      read(P, 3);
      __builtin_amdgcn_sched_barrier(0);
      // A of step s + 1 (its buffer was last read before the previous barrier)
      if (SP && s + 1 < ns) store_a(s + 1);
      mfma(2, nothing);
      if (s + 1 < ns) {
        wait_vmcnt<0>();      // this wave's copies of step s + 1
        lds_wait_barrier();   // every wave's; step s's fragments are in registers
        read(P ^ 1, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the copies of step s + 2 between the MFMAs
      mfma(3, [&](int j) __attribute__((always_inline)) {
        if (s + 2 < ns) {
          __builtin_amdgcn_sched_barrier(0);
          if (j == 0) load_a(s + 2);
          if (s + 2 < b_in) {
            TD::template issue_fast<0, TD::PER_WAVE>(cb, offB, stage_lds(P) + 2 * OPB, wave, j * TD::PER_WAVE / NH, (j + 1) * TD::PER_WAVE / NH);
            if (j == NH - 1) cb += sb;
          } else if (j == 0) {
            load_b(s + 2);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    };
    for (int s = 0; s < ns; s += 2) {
      step(std::integral_constant<int, 0>{}, s);
      if (s + 1 < ns) step(std::integral_constant<int, 1>{}, s + 1);
    }
  };

  // Unit u = (chunk, tile).  Workgroup ids go to the 8 XCDs in turn; each XCD
  // takes a contiguous range of units.
  const int units = g.ntiles * g.chunks, full = units & ~7, b = (int)blockIdx.x;
  const int u = b < full ? (b & 7) * (full >> 3) + (b >> 3) : b;
  const int chunk = u / g.ntiles, t = u - chunk * g.ntiles;
  const int s0 = (int)((int64_t)chunk * g.steps / g.chunks), s1 = (int)((int64_t)(chunk + 1) * g.steps / g.chunks);
  int q = 0;
#pragma unroll
  for (int k = 1; k < kWgradJobs; ++k)
    if (t >= g.job[k].tile0) q = k;
  const WgradJob& jb = g.job[q];
  const int64_t m0 = (int64_t)((t - jb.tile0) / jb.tiles_n) * TB, n0 = (int64_t)((t - jb.tile0) % jb.tiles_n) * TB;
  if (jb.sparse) run(std::true_type{}, jb, m0, n0, s0, s1 - s0);
  else run(std::false_type{}, jb, m0, n0, s0, s1 - s0);
  // element e of acc[i][j] in lane l: row l % 16, column 4 (l / 16) + e of its block
  float* dst = g.part + (int64_t)u * (TB * TB) + (wm * TM + (lane & 15)) * TB + wn * TN + 4 * (lane >> 4);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) *(f32x4*)(dst + i * 16 * TB + j * 16) = acc[i][j];
}

// Writes a 64 x 64 (m, n) tile of sums held as acc[i] = row m0 + ty + 16 i,
// float4 columns n0 + 4 tx: to out[m][n], or to out[n][m] when transposing
// (through LDS, so that consecutive threads store consecutive m).  N and a
// non-transposed ldo are multiples of 4 (the model dimensions are multiples
// of 8).
__device__ __forceinline__ void reduce_store(const float4 (&acc)[4], int64_t m0, int64_t n0, int tx, int ty,
                                             int64_t N, int64_t rows_out, int transpose, float* __restrict__ out,
                                             int64_t ldo, float (*tile)[65]) {
  const int64_t n = n0 + 4 * tx;
  if (!transpose) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t m = m0 + ty + 16 * i;
      if (m < rows_out && n < N) *(float4*)(out + m * ldo + n) = acc[i];
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    tile[4 * tx + 0][ty + 16 * i] = acc[i].x;
    tile[4 * tx + 1][ty + 16 * i] = acc[i].y;
    tile[4 * tx + 2][ty + 16 * i] = acc[i].z;
    tile[4 * tx + 3][ty + 16 * i] = acc[i].w;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * 64; q += 256) {
    const int r = q / 64, c = q % 64;
    const int64_t on = n0 + r, om = m0 + c;
    if (on < N && om < rows_out) out[on * ldo + om] = tile[r][c];
  }
}

// Sums the partial tiles over the chunks, in order.  One 64 x 64 block of one
// output per block.
template <int TB>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const WgradArgs g) {
  __shared__ float tile[64][65];
  int q = 0;
#pragma unroll
  for (int k = 1; k < kWgradJobs; ++k)
    if ((int)blockIdx.x >= g.job[k].rblock0) q = k;
  const WgradJob& jb = g.job[q];
  const int rb = (int)blockIdx.x - jb.rblock0;
  const int64_t m0 = (int64_t)(rb / jb.rblocks_n) * 64, n0 = (int64_t)(rb % jb.rblocks_n) * 64;
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int64_t t = jb.tile0 + (m0 / TB) * jb.tiles_n + n0 / TB;
  const float* slot = g.part + t * (TB * TB) + ((m0 % TB) + ty) * TB + (n0 % TB) + 4 * tx;
  const int64_t stride = (int64_t)g.ntiles * (TB * TB);
  float4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  // four chunks at a time (16 loads in flight per thread), added in order
  for (int c = 0; c < g.chunks; c += 4) {
    float4 v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[u][i] = c + u < g.chunks ? *(const float4*)(slot + (c + u) * stride + i * 16 * TB) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[i].x += v[u][i].x; acc[i].y += v[u][i].y; acc[i].z += v[u][i].z; acc[i].w += v[u][i].w;
      }
  }
  reduce_store(acc, m0, n0, tx, ty, jb.N, jb.rows_out, jb.transpose, jb.out, jb.ldo, tile);
}

}  // namespace elas
