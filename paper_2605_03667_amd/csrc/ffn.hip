// Launch sequences of the ELAS low-rank 2:4 FFN on one GPU: forward (ELAS
// Fig. 1 caption; Eq. 1-3, Algorithm 1), backward (Sec. 3.3.2, Sec. 3.4) and
// the standalone 2:4 sparse x dense product.  Everything runs on the caller's
// stream in the caller's workspace; nothing here allocates.
#include <algorithm>
#include <atomic>

#include "gemm.h"
#include "internal.h"
#include "plain.h"
#include "resident.h"
#include "small.h"
#include "wgrad.h"

namespace elas {

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t n) { return (n + kAlign - 1) / kAlign * kAlign; }
int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Carves consecutive aligned regions out of the caller's workspace.
struct Carver {
  char* p;
  size_t used = 0;
  template <class T>
  T* take(size_t count) {
    T* r = p ? (T*)(p + used) : nullptr;
    used += align_up(count * sizeof(T));
    return r;
  }
};

// ---- small kernels -----------------------------------------------------------

// Transposing job: out[j][i] = in[i][j] for i < rows, j < cols; 0 elsewhere
// in [out_rows x out_cols].  Copying job (transpose = 0): out[i][j] = in[i][j],
// 0 elsewhere.  The output is row-major with pitch ldo, blocked (blocked_index)
// when nsk > 0, or in fragment order (frag_index) when kp > 0.
struct TransposeJob {
  const uint16_t* in;
  uint16_t* out;
  int64_t rows, cols, ldi, out_rows, out_cols, ldo;
  int tiles_x;      // 64-wide tiles along out_cols
  int tile_begin;   // first flat tile index of this job
  int transpose;
  int64_t nsk;
  int64_t kp;       // K panels of the fragment order
};
__device__ __forceinline__ int64_t job_pos(const TransposeJob& jb, int64_t row, int64_t col) {
  if (jb.kp > 0) return frag_index(row, col, jb.kp);
  return jb.nsk > 0 ? blocked_index(row, col, jb.nsk) : row * jb.ldo + col;
}
// Up to four jobs in one launch (the weight factors of one call): the flat tile
// index selects the job, so small factors share the launch.
constexpr int kMaxTransposeJobs = 4;
struct TransposeBatch {
  TransposeJob job[kMaxTransposeJobs];
  int n;
};

__global__ __launch_bounds__(256) void transpose_pad_kernel(TransposeBatch tb) {
  // 64 x 64 tile, moved in 16-byte pieces (8 bf16): thread t reads row
  // i0 + t/8 (+32) at columns j0 + 8 (t%8), and writes output row j0 + t/8
  // (+32) at columns i0 + 8 (t%8).  cols, ldi, out_cols and ldo are
  // multiples of 8 (model dimensions), so a piece is wholly inside or outside.
  // The LDS rows are padded to 72 elements so that the column reads of the
  // write phase fall in distinct banks.
  __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];
  int q = 0;
#pragma unroll
  for (int k = 1; k < kMaxTransposeJobs; ++k)
    if (k < tb.n && (int)blockIdx.x >= tb.job[k].tile_begin) q = k;
  const TransposeJob& jb = tb.job[q];
  const int t = (int)blockIdx.x - jb.tile_begin;
  const int r = threadIdx.x / 8, c = threadIdx.x % 8;
  if (!jb.transpose) {   // (uniform over the workgroup: one job per tile)
    const int64_t r0 = (int64_t)(t / jb.tiles_x) * 64, c0 = (int64_t)(t % jb.tiles_x) * 64;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t i = r0 + r + 32 * h, j = c0 + 8 * c;
      if (i < jb.out_rows && j < jb.out_cols) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (i < jb.rows && j < jb.cols) v = *(const uint4*)(jb.in + i * jb.ldi + j);
        *(uint4*)(jb.out + job_pos(jb, i, j)) = v;
      }
    }
    return;
  }
  const int64_t i0 = (int64_t)(t % jb.tiles_x) * 64, j0 = (int64_t)(t / jb.tiles_x) * 64;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a = r + 32 * h;
    const int64_t i = i0 + a, j = j0 + 8 * c;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (i < jb.rows && j < jb.cols) v = *(const uint4*)(jb.in + i * jb.ldi + j);
    *(uint4*)&tile[a][8 * c] = v;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a = r + 32 * h;                       // output row j0 + a = input column
    const int64_t jj = j0 + a, ii = i0 + 8 * c;
    if (jj < jb.out_rows && ii < jb.out_cols) {
      uint32_t w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = (uint32_t)tile[8 * c + 2 * k][a] | ((uint32_t)tile[8 * c + 2 * k + 1][a] << 16);
      *(uint4*)(jb.out + job_pos(jb, jj, ii)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// Collects transposes and launches them together.
struct Transposes {
  TransposeBatch tb{};
  int tiles = 0;
  void add(const uint16_t* in, int64_t rows, int64_t cols, int64_t ldi, uint16_t* out, int64_t out_rows,
           int64_t out_cols, int64_t ldo, int transpose = 1, int64_t nsk = 0, int64_t kp = 0) {
    TransposeJob& j = tb.job[tb.n++];
    j = TransposeJob{in, out, rows, cols, ldi, out_rows, out_cols, ldo, (int)cdiv(out_cols, 64), tiles, transpose, nsk, kp};
    tiles += j.tiles_x * (int)cdiv(out_rows, 64);
  }
  hipError_t launch(hipStream_t st) {
    if (tiles == 0) return hipSuccess;
    TimedLaunch tl("weight_transpose", st);
    hipLaunchKernelGGL(transpose_pad_kernel, dim3((unsigned)tiles), dim3(256), 0, st, tb);
    return hipGetLastError();
  }
};

hipError_t transpose_pad(const uint16_t* in, int64_t rows, int64_t cols, int64_t ldi, uint16_t* out,
                         int64_t out_rows, int64_t out_cols, int64_t ldo, hipStream_t st) {
  Transposes t;
  t.add(in, rows, cols, ldi, out, out_rows, out_cols, ldo);
  return t.launch(st);
}

// bf16 result of a split-K product with a bf16 output: out[m][n] =
// bf16(sum over the splits k, in order, of part[k][m][n]); one 4-column piece
// per thread (N and ldo are multiples of 8).
__global__ __launch_bounds__(256) void splitk_reduce_bf16_kernel(const float* __restrict__ part, int splits, int64_t M,
                                                                int64_t N, uint16_t* __restrict__ out, int64_t ldo) {
  const int64_t pieces = N / 4;
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= M * pieces) return;
  const int64_t m = q / pieces, n = (q % pieces) * 4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k = 0; k < splits; ++k) {
    const float4 v = *(const float4*)(part + ((int64_t)k * M + m) * N + n);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  *(uint2*)(out + m * ldo + n) = make_uint2(bf16x2_rne(acc.x, acc.y), bf16x2_rne(acc.z, acc.w));
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) p[e] = 0.f;
}

hipError_t fill_zero(float* p, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  TimedLaunch tl("fill_zero", st);
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

// ---- GEMM configurations -----------------------------------------------------
// Tile shapes picked by measurement on MI355X at the 1B FFN shapes: eight
// waves (two per SIMD) hide LDS and global latency better than four larger
// wave tiles.
// Dense products with both operands K-contiguous: 256 x BN tiles, 4 x 2 waves.
template <int BN, int EPI, bool M_FAST, bool DEEP = false>
using CfgNT = GemmCfg<256, BN, 4, 2, OP_K, OP_K, EPI, M_FAST, 2, 128, DEEP>;
// 2:4 sparse A (smfmac) times K-contiguous B: 256 x 256 tiles, 4 x 2 waves
// (64 x 128 per wave), 64 dense K per step in three LDS stages (150 KB).  The
// full-width N tile halves the re-reads of the compressed operand, which
// streams from HBM, and the third stage covers more of its latency.
// (Measured: 22% faster than 256 x 128 tiles with 128-K steps in two stages.)
using CfgSP = GemmCfg<256, 256, 4, 2, OP_SP, OP_K, EPI_BF16, false, 3, 64>;
// Compute units of the current device (cached per device id).
// (Relaxed atomics: concurrent first calls store the same value.)
int device_cus() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

template <class Cfg>
hipError_t launch(const char* tag, GemmArgs g, int splits, hipStream_t st) {
  if (g.b_nsk > 0 && (!Cfg::B_BLOCKABLE || g.ldb != 64)) return hipErrorInvalidValue;
  g.tiles_m = (int)cdiv(g.M, Cfg::BM);
  g.tiles_n = (int)cdiv(g.N, Cfg::BN);
  if (splits <= 1) {
    splits = 1;
    g.k_split = cdiv(g.K, Cfg::BK) * Cfg::BK;
  }
  // Direct-staged kernels are persistent: one workgroup per CU at most, each
  // looping over its tiles.
  const int tiles = g.tiles_m * g.tiles_n;
  const int cus = device_cus();
  const int slots = cus * (Cfg::LDS_BYTES <= 80 * 1024 ? 2 : 1);
  const int wgs = tiles > slots ? slots : tiles;
  const dim3 grid((unsigned)wgs, (unsigned)splits);
  TimedLaunch tl(tag, st);
  hipLaunchKernelGGL(gemm_kernel<Cfg>, grid, dim3(Cfg::NT), 0, st, g);
  return hipGetLastError();
}

// Dense products (plain.h): 256 x 256 tiles on 8 waves with the streaming operand
// three steps deep, 256 x 128 for narrow outputs; 128 x 128 on 4 waves, two
// workgroups per CU.
template <int EPI>
using PlainNT = PlainCfg<256, 256, 4, 2, EPI, 3, 2>;
template <int EPI>
using PlainNTn = PlainCfg<256, 128, 4, 2, EPI, 3, 3>;
template <int EPI>
using PlainNTs = PlainCfg<128, 128, 2, 2, EPI, 3, 2>;

template <class Cfg>
hipError_t launch_plain(const char* tag, GemmArgs g, int splits, hipStream_t st) {
  if (g.b_nsk > 0 && g.ldb != 64) return hipErrorInvalidValue;
  g.tiles_m = (int)cdiv(g.M, Cfg::BM);
  g.tiles_n = (int)cdiv(g.N, Cfg::BN);
  if (splits <= 1) {
    splits = 1;
    g.k_split = cdiv(g.K, Cfg::BK) * Cfg::BK;
  }
  const int tiles = g.tiles_m * g.tiles_n, slots = device_cus() * (Cfg::LDS <= 80 * 1024 ? 2 : 1);
  TimedLaunch tl(tag, st);
  hipLaunchKernelGGL(plain_kernel<Cfg>, dim3((unsigned)std::min(tiles, slots), (unsigned)splits), dim3(Cfg::NT), 0, st, g);
  return hipGetLastError();
}

// Small problems: when 256-wide tiles would leave more than a quarter of the
// CUs without a tile, 128 x 128 tiles (4 waves of 64 x 64) give four times as
// many (twice as many for the staged 2:4 epilogues, which need 256 features).
// In between: 256 x 128 tiles on 8 waves (64 x 64 per wave), four stages (136 KB).
using CfgSPn = GemmCfg<256, 128, 4, 2, OP_SP, OP_K, EPI_BF16, false, 4, 64>;
// Row-layout operands (elas_spmm_24): 128 K per step in two stages (136 KB), so that a
// row's kept values come 128 bytes at a time, a cache line, and not 64.
using CfgSPr = GemmCfg<256, 128, 4, 2, OP_SP, OP_K, EPI_BF16, false, 2, 128>;
using CfgSPs = GemmCfg<128, 128, 2, 2, OP_SP, OP_K, EPI_BF16, false, 3, 64>;

bool few_tiles(int64_t M, int64_t N, int bm, int bn) { return cdiv(M, bm) * cdiv(N, bn) * 4 < 3LL * device_cus(); }

// Split-K of a bf16-output product with few 128 x 128 tiles and a long K:
// enough splits to cover the CUs once, each at least 8 K steps of bk; the fp32
// partials [splits x M x N] are then summed in split order and rounded once.
struct SmallSplit {
  int splits;
  int64_t k_split;
};
SmallSplit plan_small_split(int64_t M, int64_t N, int64_t K, int bk) {
  const int64_t tiles = cdiv(M, 128) * cdiv(N, 128), cus = device_cus();
  const int64_t steps = cdiv(K, bk);
  if (tiles == 0 || tiles * 2 > cus || steps < 16) return {1, K};   // (no rows: nothing to split)
  int64_t s = cus / tiles;
  if (s > steps / 8) s = steps / 8;
  if (s < 2) return {1, K};
  const int64_t k_split = cdiv(cdiv(K, s), bk) * bk;
  return {(int)cdiv(K, k_split), k_split};
}
size_t small_split_bytes(int64_t M, int64_t N, int64_t K, int bk) {
  const SmallSplit p = plan_small_split(M, N, K, bk);
  return p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
}
template <int EPI, bool M_FAST>
using CfgNTs = GemmCfg<128, 128, 2, 2, OP_K, OP_K, EPI, M_FAST>;
using CfgSPsf = GemmCfg<128, 128, 2, 2, OP_SP, OP_K, EPI_F32, false, 3, 64>;

hipError_t reduce_bf16(const float* part, int splits, int64_t M, int64_t N, uint16_t* out, int64_t ldo,
                       hipStream_t st) {
  TimedLaunch tl("splitk_reduce_bf16", st);
  hipLaunchKernelGGL(splitk_reduce_bf16_kernel, dim3((unsigned)cdiv(M * (N / 4), 256)), dim3(256), 0, st, part, splits,
                     M, N, out, ldo);
  return hipGetLastError();
}

// 2:4 A times K-contiguous B, bf16 out (`part`: split-K partials, may be null).
hipError_t launch_sp(const char* tag, GemmArgs g, hipStream_t st, float* part = nullptr) {
  if (few_tiles(g.M, g.N, 256, 256)) {
    const SmallSplit p = part ? plan_small_split(g.M, g.N, g.K, CfgSPsf::BK) : SmallSplit{1, g.K};
    if (p.splits > 1) {
      uint16_t* out = (uint16_t*)g.C;
      const int64_t ldo = g.ldc;
      g.C = part;
      g.ldc = g.N;
      g.k_split = p.k_split;
      hipError_t e = launch<CfgSPsf>(tag, g, p.splits, st);
      if (e != hipSuccess) return e;
      return reduce_bf16(part, p.splits, g.M, g.N, out, ldo, st);
    }
  }
  // Microseconds per K step of one round of tiles (measured at 86 steps: 256 x 256
  // 215 us in two rounds, 256 x 128 86 us, 128 x 128 99 us with two workgroups per
  // CU and 44 us with one): the tiling with the least total.  Of a row-layout operand the
  // 256 x 128 tiles with 128-K steps take 0.8 (us at 5464 x 512, with 64-K steps, with
  // these, 256 x 256, 128 x 128: 16384 rows 98, 77, 107, -; 65536 rows 401, 349, 300, -;
  // 4096 rows 74, 62, 105, 53).
  const int64_t cus = device_cus(), t128 = cdiv(g.M, 128) * cdiv(g.N, 128), last = t128 % (2 * cus);
  const double big = 1.25 * cdiv(cdiv(g.M, 256) * cdiv(g.N, 256), cus), mid = (g.a_tiled ? 1.0 : 0.8) * cdiv(cdiv(g.M, 256) * cdiv(g.N, 128), cus);
  const double small = 1.15 * (t128 / (2 * cus)) + (last == 0 ? 0.0 : last <= cus ? 0.51 : 1.15);
  if (small < mid && small < big) return launch<CfgSPs>(tag, g, 1, st);
  if (mid < big) return g.a_tiled ? launch<CfgSPn>(tag, g, 1, st) : launch<CfgSPr>(tag, g, 1, st);
  return launch<CfgSP>(tag, g, 1, st);
}
// Epilogues that select and compress 2:4 groups (features along M).
// With more than 3 MB of A rows (the d_ff-wide weight factor: 5.6 MB at 1B,
// beyond an XCD's 4 MB L2) and an even number of 256-row tiles, two panels.
template <int EPI>
hipError_t launch_staged(const char* tag, GemmArgs g, hipStream_t st) {
  if (few_tiles(g.M, g.N, 256, 256)) return launch<CfgNT<128, EPI, true>>(tag, g, 1, st);
  const int64_t tiles_m = cdiv(g.M, 256);
  if (tiles_m % 2 == 0 && tiles_m * 256 * g.K * 2 > (int64_t(3) << 20)) g.m_groups = 2;
  return launch<CfgNT<256, EPI, true>>(tag, g, 1, st);
}
// Epilogues that write the dense dH (features along M).
template <int EPI>
hipError_t launch_act(const char* tag, const GemmArgs& g, hipStream_t st) {
  if (few_tiles(g.M, g.N, 256, 256)) return launch<CfgNTs<EPI, true>>(tag, g, 1, st);
  return launch<CfgNT<256, EPI, true, true>>(tag, g, 1, st);
}

// Token-resident products (resident.h), for the ranks it is compiled for: those of the
// model shapes (its LDS block and registers would hold any multiple of 64 up to 512).
bool resident_rank(int64_t r) { return r == 128 || r == 256 || r == 512; }
// The d_ff-wide ones (up projection and dH) are faster than the tiled kernel at
// every token count (microseconds, tiled against this: 60M at 512 tokens k2
// 10.0 / 8.6, b3 11.6 / 9.5; 1B at 2048 29.5 / 21.3, 33.5 / 22.3; 1B at 65536
// 424 / 307, 478 / 334), but where nothing else is laid out in the call, laying
// the weights out in fragment order is a launch of its own.  It pays for itself from
// 2049 tokens, unless the tiled kernel has them all in one round of tiles (at r = 256
// in a full one); at dense activations from about 12 G multiplications.  Whole
// forwards with the factors as a linear layer stores them, us, both products tiled
// against this with its layout (and Y, below, as it is there): 60M at 4096 tokens
// 30.8 / 32.5, at 8192 43.9 / 45.7, at 12000 55.5 / 53.5; 130M at 4096 45.0 / 50.7, at
// 6000 57.3 / 56.1, at 8192 58.9 / 60.8, at 16384 82.2 / 78.1; 350M at 3000 56.8 / 54.3;
// 1B at 2049 84.2 / 77.4; dense 60M at 8192 43.1 / 46.5, 130M at 16384 81.8 / 84.9 and at
// 32768 140 / 135, 350M at 16384 103 / 107 and at 32768 200 / 191, 1B at 4096
// 116 / 122 and at 6000 162 / 158.
bool own_layout_pays(int64_t T, int64_t F, int64_t r, bool dense) {
  if (T <= 2048) return false;
  const int64_t Fp = pad64(F), cus = device_cus();
  if (dense) return (double)T * Fp * r > 1.2e10;
  const int64_t tiles = cdiv(Fp, 256) * cdiv(T, few_tiles(Fp, T, 256, 256) ? 128 : 256);   // of launch_staged
  const bool one_round = r <= 128 ? tiles <= cus : r <= 256 && tiles <= cus && 8 * tiles > 7 * cus;
  return !one_round;
}
bool resident_wide(int64_t T, int64_t F, int64_t r, bool dense, bool laid_out) {
  return resident_rank(r) && T > 0 && (laid_out || own_layout_pays(T, F, r, dense));
}
// The d-wide ones (Y and dx), whose few features leave a split-K or 128-wide
// tiling ahead up to 4096 tokens (whole forwards, tiled / this: 60M at 4096 31.6 / 32.5,
// 130M 47.9 / 50.7, 350M 57.6 / 58.6, 1B 105.4 / 108.5; at 32768 70.8 / 70.8,
// 122 / 117, 161 / 159, 460 / 454; training steps of 4096 1.5 to 0 % less tiled).
bool resident_down(int64_t T, int64_t r) { return resident_rank(r) && T > 4096; }
// Workgroups per block of 128 tokens: the split of the nfb 64-feature blocks
// with the fewest rounds of wave tiles (copying the tokens costs about 0.4 of
// one).
int resident_split(int64_t tiles, int64_t nfb, int64_t nw) {
  const int64_t slots = device_cus() * (8 / nw);
  int best = 1;
  double best_cost = 1e30;
  for (int64_t s = 1; s <= nfb && s <= 16; ++s) {
    const double cost = (double)cdiv(tiles * s, slots) * (0.4 + (double)cdiv(cdiv(nfb, s), nw));
    if (cost < best_cost * 0.98) { best_cost = cost; best = (int)s; }
  }
  return best;
}
template <int EPI>
hipError_t launch_resident(const char* tag, int64_t r, ResArgs g, hipStream_t st) {
  const int64_t tiles = cdiv(g.T, 128);
  const int nw = res_waves(EPI, (int)(r / 64));
  g.fsplit = resident_split(tiles, g.nfb, nw);
  TimedLaunch tl(tag, st);
  const dim3 grid((unsigned)(tiles * g.fsplit));
  if (r == 128)
    hipLaunchKernelGGL((resident_kernel<EPI, 2>), grid, dim3(64 * nw), 0, st, g);
  else if (r == 256)
    hipLaunchKernelGGL((resident_kernel<EPI, 4>), grid, dim3(64 * nw), 0, st, g);
  else
    hipLaunchKernelGGL((resident_kernel<EPI, 8>), grid, dim3(64 * nw), 0, st, g);
  return hipGetLastError();
}
// C [T x M] = X W^T with W [M x r] in fragment order.
hipError_t resident_bf16(const char* tag, const uint16_t* W, const uint16_t* X, int64_t T, int64_t M, int64_t r, uint16_t* C,
                         hipStream_t st) {
  ResArgs g{};
  g.W = W; g.X = X; g.ldx = r; g.T = T; g.nfb = (int)(pad64(M) / 64); g.C = C; g.ldc = M; g.f_valid = (int)M;
  return launch_resident<EPI_BF16>(tag, r, g, st);
}

// Wave-split products (small.h).
template <int EPI, bool SP, int TT, int FI, int FW, int D, int MAXW>
hipError_t launch_small_as(const char* tag, const SmallArgs& g, hipStream_t st) {
  const int waves = g.ks * FW;
  const size_t lds = (size_t)waves * FI * TT * 1024;
  if (waves > MAXW || lds > 64 * 1024) return hipErrorInvalidValue;
  TimedLaunch tl(tag, st);
  const dim3 grid((unsigned)cdiv(g.M, FW * FI * 16), (unsigned)cdiv(g.T, TT * 16));
  hipLaunchKernelGGL((small_kernel<EPI, SP, TT, FI, FW, D, MAXW>), grid, dim3(64 * waves), lds, st, g);
  return hipGetLastError();
}
// Sums cut as the tiled product's split-K cuts them (one chunk where it is not split).
SmallSplit tiled_chunks(int64_t T, int64_t M, int64_t K) {
  return few_tiles(T, M, 256, 256) ? plan_small_split(T, M, K, 64) : SmallSplit{1, K};
}
// Long contractions (over d or d_ff) to M features, one wave per chunk of K.  Blocks
// per wave: the fewest with which each CU has at most one workgroup, or two where
// those are of few waves; with more the tiled kernel is ahead, and earlier where there
// are many chunks.  Whole calls in us, tiled against 1 x 1, 2 x 1, 2 x 2, 4 x 1 and
// 4 x 2 (token x feature) blocks:
//   forward, k1:   60M, 1 chunk,  2048 tokens  34.9 | 33.2  32.6  31.5  33.5  33.4
//                  350M, 2,       2000         47.7 | 50.6  47.1  44.3  45.6  43.4
//                  1B, 4,         16           36.2 | 31.7  31.9  33.6  33.0  34.8
//                                 256          52.7 | 49.2  47.3  49.2  50.9  53.0
//                                 512          56.9 | 58.8  55.4  52.1  53.9  56.1
//                                 1024         60.8 | 76.3  69.6  62.8  66.2  59.6
//   forward, k3:   60M, 2,        4096         42.3 | 40.1  37.8  35.7  37.5  37.7
//                  350M, 5,       2000         47.7 | 56.5  49.2  46.7  46.1  43.3
//                  1B, 10,        512          56.9 | 67.0  55.9    -   52.4    -
//                  1B, 8,         1024         60.8 | 84.8  71.8  67.8  66.2  61.3
//   dense step, k3: 60M, 2,       2048         99.5 | 95.8  95.0  93.0  95.7  95.4
//                  1B, 8,         1000        183.2 | 220   209   197   203   191
//   the same and b5: 1B, 10,      512         156   |  -     -     -    150     -
// 0: the tiled kernel; else the shape of launch_small_long.
template <bool SP>
int small_long_shape(int64_t T, int64_t M, const SmallSplit& p) {
  if (T <= 0 || p.splits > 16) return 0;
  const int64_t cus = device_cus(), m1 = cdiv(M, 16), m2 = cdiv(M, 32);
  const int64_t most = p.splits <= (SP || M <= 128 ? 2 : 1) ? 2 * cus : cus;
  if (m1 * cdiv(T, 16) <= most) return 1;
  if (m1 * cdiv(T, 32) <= cus) return 2;
  if (p.splits <= (SP ? 2 : 8) && m2 * cdiv(T, 32) <= most) return 3;
  if (p.splits > (SP ? 2 : 8) && p.splits <= 12 && m1 * cdiv(T, 64) <= cus) return 4;
  return p.splits <= 6 && m2 * cdiv(T, 64) <= cus ? 5 : 0;
}
template <bool SP>
hipError_t launch_small_long(const char* tag, SmallArgs g, const SmallSplit& p, hipStream_t st) {
  g.ks = p.splits;
  g.chunk = (int)cdiv(p.k_split, 64);
  switch (small_long_shape<SP>(g.T, g.M, p)) {
    case 1:   // (a lone wave row of few chunks: all of a short K in flight; 60M, 16 tokens, k3 18.4 -> 18.1)
      if (p.splits <= 8 && cdiv(g.M, 16) * cdiv(g.T, 16) <= device_cus()) return launch_small_as<EPI_BF16, SP, 1, 1, 1, 8, 8>(tag, g, st);
      return launch_small_as<EPI_BF16, SP, 1, 1, 1, 4, 16>(tag, g, st);
    case 2: return launch_small_as<EPI_BF16, SP, 2, 1, 1, 3, 16>(tag, g, st);
    case 3: return launch_small_as<EPI_BF16, SP, 2, 2, 1, 3, 8>(tag, g, st);
    case 4: return launch_small_as<EPI_BF16, SP, 4, 1, 1, 3, 12>(tag, g, st);
    case 5: return launch_small_as<EPI_BF16, SP, 4, 2, 1, 2, 8>(tag, g, st);
    default: return hipErrorInvalidValue;
  }
}
// Short ones (over r): features over the waves, each with the whole of K, by the same
// measure (k2 at 1B, 64 tokens 19.0 / 10.6; k4 at 1B, 256 tokens 11.4 / 9.9; k4 at
// 350M, 500 tokens 10.4 / 7.3).
bool small_short(int64_t T, int64_t M) { return T > 0 && cdiv(M, 64) * cdiv(T, 32) <= device_cus(); }
// (plain output, where the tiled kernel may cut K = r)
bool small_short(int64_t T, int64_t M, int64_t K) { return small_short(T, M) && tiled_chunks(T, M, K).splits == 1; }
template <int EPI>
hipError_t launch_small_short(const char* tag, SmallArgs g, hipStream_t st) {
  g.ks = 1;
  g.chunk = (int)cdiv(g.K, 64);
  if (g.T <= 16) return launch_small_as<EPI, false, 1, 1, 4, 8, 4>(tag, g, st);
  return launch_small_as<EPI, false, 2, 1, 4, 4, 4>(tag, g, st);
}
// C [T x M] = X W^T, W [M x K].
SmallArgs small_dense(const uint16_t* W, int64_t ldw, int64_t M, int64_t K, const uint16_t* X, int64_t ldx, int64_t T, uint16_t* C) {
  SmallArgs g{};
  g.W = W; g.ldw = ldw; g.m_valid = g.M = (int)M; g.kw_valid = g.K = (int)K;
  g.X = X; g.ldx = ldx; g.T = T; g.C = C; g.ldc = M;
  return g;
}
// C [T x M] = S W^T with S compressed (tiled) along K = F features, W [M x ldw].
SmallArgs small_sp(const uint16_t* W, int64_t ldw, int64_t M, int64_t F, const uint16_t* sv, const uint8_t* sm, int64_t T, uint16_t* C) {
  SmallArgs g{};
  g.W = W; g.ldw = ldw; g.m_valid = g.M = (int)M; g.kw_valid = (int)F; g.K = (int)pad64(F);
  g.X = sv; g.Xm = sm; g.ldx = vals_ld(F); g.ldxm = meta_ld(F); g.T = T; g.C = C; g.ldc = M;
  return g;
}
// Y and dx.
hipError_t launch_small_down(const char* tag, const SmallArgs& g, hipStream_t st) {
  const SmallSplit p = tiled_chunks(g.T, g.M, g.K);
  return p.splits == 1 ? launch_small_short<EPI_BF16>(tag, g, st) : launch_small_long<false>(tag, g, p, st);
}
// The kernel of each product of one call.
enum Route { TILED, SMALL, RESIDENT };
// P and dZ (K = d); Z and dP (K = d_ff, padded to 64 where the activation is compressed).
template <bool SP>
Route route_long(int64_t T, int64_t M, int64_t K) { return small_long_shape<SP>(T, M, tiled_chunks(T, M, K)) ? SMALL : TILED; }
Route route_over_ff(int64_t T, int64_t F, int64_t r, bool sp) { return sp ? route_long<true>(T, r, pad64(F)) : route_long<false>(T, r, F); }
// The up projection and masked dH (sparse mode) or their dense counterparts;
// laid_out: the call lays out weights anyway.
Route route_wide(int64_t T, int64_t F, int64_t r, bool dense, bool laid_out) {
  if (!dense && small_short(T, pad64(F))) return SMALL;
  return resident_wide(T, F, r, dense, laid_out) ? RESIDENT : TILED;
}
// Y and dx.
Route route_down(int64_t T, int64_t d, int64_t r) {
  if (small_short(T, d, r) || (tiled_chunks(T, d, r).splits > 1 && route_long<false>(T, d, r) == SMALL)) return SMALL;
  return resident_down(T, r) ? RESIDENT : TILED;
}

// Dense product C[M x N] = A[M x K] * Bt[N x K]^T in bf16, or relu(.)^2 of it
// (`part`: split-K partials for small problems of EPI_BF16, may be null).
// b_nsk > 0: Bt is blocked (blocked_index, b_nsk K blocks per panel; ldb is
// then ignored).
template <int EPI>
hipError_t gemm_nt(const char* tag, const uint16_t* A, int64_t lda, const uint16_t* Bt, int64_t ldb, uint16_t* C, int64_t ldc,
                        int64_t M, int64_t N, int64_t K, hipStream_t st, float* part = nullptr, int64_t b_nsk = 0) {
  GemmArgs g{};
  g.A = A; g.lda = lda; g.B = Bt; g.ldb = b_nsk > 0 ? 64 : ldb; g.b_nsk = b_nsk; g.C = C; g.ldc = ldc;
  g.M = M; g.N = N; g.K = K; g.m_valid = M; g.ka_valid = K; g.kb_valid = K;
  if (few_tiles(M, N, 256, N <= 128 ? 128 : 256)) {
    const SmallSplit p = part ? plan_small_split(M, N, K, 64) : SmallSplit{1, K};
    if (p.splits > 1) {
      g.C = part;
      g.ldc = N;
      g.k_split = p.k_split;
      const hipError_t e = launch_plain<PlainNTs<EPI_F32>>(tag, g, p.splits, st);
      if (e != hipSuccess) return e;
      return reduce_bf16(part, p.splits, M, N, C, ldc, st);
    }
    return launch_plain<PlainNTs<EPI>>(tag, g, 1, st);
  }
  if (N <= 128) return launch_plain<PlainNTn<EPI>>(tag, g, 1, st);
  return launch_plain<PlainNT<EPI>>(tag, g, 1, st);
}
hipError_t gemm_nt_bf16(const char* tag, const uint16_t* A, int64_t lda, const uint16_t* Bt, int64_t ldb, uint16_t* C, int64_t ldc,
                        int64_t M, int64_t N, int64_t K, hipStream_t st, float* part = nullptr, int64_t b_nsk = 0) {
  return gemm_nt<EPI_BF16>(tag, A, lda, Bt, ldb, C, ldc, M, N, K, st, part, b_nsk);
}

// Weight gradients (wgrad.h): the jobs of one backward and how their (tile, step)
// list is shared out.
struct WgradPlan {
  WgradArgs g{};
  int tb = 0, njobs = 0, rblocks = 0;
  void add(const uint16_t* A, int64_t lda, const uint8_t* Am, int64_t ldam, const uint16_t* B, int64_t M, int64_t N,
           float* out, int64_t rows_out, bool transpose) {
    WgradJob& j = g.job[njobs++];
    j = WgradJob{};
    j.A = A; j.lda = lda; j.Am = Am; j.ldam = ldam; j.sparse = Am != nullptr;
    j.B = B; j.ldb = N; j.M = M; j.N = N;
    j.out = out; j.rows_out = rows_out; j.transpose = transpose; j.ldo = transpose ? rows_out : N;
  }
  // 256-wide tiles as long as each of one workgroup per CU gets about 6 steps;
  // else 128-wide ones, two workgroups per CU, at least 4 steps each (fewer steps
  // than that cost more in partial tiles than the extra workgroups give).
  void finish(int64_t T) {
    const int64_t steps = cdiv(T, 64), cus = device_cus();
    auto tiles = [&](int b) {
      int64_t n = 0;
      for (int k = 0; k < njobs; ++k) n += cdiv(g.job[k].M, b) * cdiv(g.job[k].N, b);
      return n;
    };
    tb = tiles(256) * steps >= 6 * cus ? 256 : 128;
    int64_t nt = 0;
    for (int k = 0; k < kWgradJobs; ++k) {
      WgradJob& j = g.job[k];
      j.tile0 = (int)nt;
      j.rblock0 = rblocks;
      if (k >= njobs) {   // never reached
        j.tile0 = j.rblock0 = INT32_MAX;
        continue;
      }
      j.tiles_n = (int)cdiv(j.N, tb);
      j.rblocks_n = (int)cdiv(j.N, 64);
      nt += cdiv(j.M, tb) * j.tiles_n;
      rblocks += j.rblocks_n * (int)cdiv(j.rows_out, 64);
    }
    const int64_t slots = tb == 256 ? cus : 2 * cus;
    int64_t c = std::min(slots / nt, tb == 256 ? steps : steps / 4);
    if (c < 1) c = 1;
    g.T = T;
    g.steps = (int)steps;
    g.ntiles = (int)nt;
    g.chunks = (int)c;
  }
  size_t part_floats() const { return (size_t)g.ntiles * g.chunks * tb * tb; }
  hipError_t launch(const char* tag, hipStream_t st) const {
    {
      TimedLaunch tl(tag, st);
      if (tb == 256) hipLaunchKernelGGL(wgrad_kernel<256>, dim3((unsigned)(g.ntiles * g.chunks)), dim3(512), 0, st, g);
      else hipLaunchKernelGGL(wgrad_kernel<128>, dim3((unsigned)(g.ntiles * g.chunks)), dim3(256), 0, st, g);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    TimedLaunch tl("wgrad_reduce", st);
    if (tb == 256) hipLaunchKernelGGL(wgrad_reduce_kernel<256>, dim3((unsigned)rblocks), dim3(256), 0, st, g);
    else hipLaunchKernelGGL(wgrad_reduce_kernel<128>, dim3((unsigned)rblocks), dim3(256), 0, st, g);
    return hipGetLastError();
  }
};

struct FwdWs {
  uint16_t *U_upT, *V_upT, *U_downT, *V_downT;
  float* part;   // split-K partials of the long-K products at small token counts
  size_t bytes;
};
// The forward's kernels over K = r.  lean: without the token-resident ones, whose
// factors in fragment order may not fit a workspace of a fixed size.
Route fwd_up(int64_t T, int64_t F, int64_t r, bool dense, bool ab, bool lean) {
  const Route w = route_wide(T, F, r, dense, !ab);
  return lean && w == RESIDENT ? TILED : w;
}
// (a layout launch for Y alone does not pay)
Route fwd_down(int64_t T, int64_t d, int64_t r, bool lean, bool ab, Route up) {
  const Route w = route_down(T, d, r);
  return (lean || (ab && up != RESIDENT)) && w == RESIDENT ? TILED : w;
}
// (ab: the caller passes the factors K-contiguous; copied for the token-resident products only)
FwdWs fwd_ws(char* p, int64_t T, int64_t d, int64_t F, int64_t r, bool dense, bool ab, bool lean) {
  const int64_t Fp = pad64(F);
  const Route up = fwd_up(T, F, r, dense, ab, lean), down = fwd_down(T, d, r, lean, ab, up);
  Carver c{p};
  FwdWs w{};
  if (!ab) {
    w.U_upT = c.take<uint16_t>(r * d);
    w.U_downT = c.take<uint16_t>(r * Fp);
  }
  // (fragment order for the token-resident products, also from A and B)
  if (!ab || up == RESIDENT) w.V_upT = c.take<uint16_t>(Fp * r);
  if (!ab || down == RESIDENT) w.V_downT = c.take<uint16_t>((down == RESIDENT ? pad64(d) : d) * r);
  size_t pb = small_split_bytes(T, r, d, 64);                 // k1
  pb = std::max(pb, small_split_bytes(T, r, Fp, 64));          // k3 (2:4 or dense)
  pb = std::max(pb, small_split_bytes(T, d, r, 64));           // k4
  w.part = pb ? c.take<float>(pb / sizeof(float)) : nullptr;
  w.bytes = c.used;
  return w;
}

// The tiled products of the backward take V_up and V_down laid out.
bool bwd_lays_out(int64_t T, int64_t d, int64_t F, int64_t r, bool dense, bool ste) {
  return route_long<false>(T, r, d) == TILED || route_over_ff(T, F, r, !dense && !ste) == TILED;
}
struct BwdWs {
  uint16_t *dZ, *dH, *dP, *V_upT;
  uint16_t *U_downR, *U_upR;   // U_down and U_up in fragment order (token-resident products)
  uint16_t *V_upB, *V_downB;   // V_up [r x F] and V_down [r x d] blocked (the B operands of b5, b1)
  float* part;
  size_t bytes;
};
// dV_down = Z^T dY; dU_down = S^T dZ from the compressed (or dense) S; dV_up =
// P^T dH as dV_up^T = dH^T P, written transposed; dU_up = x^T dP.
WgradPlan wgrad_plan(const FfnArgs& a, const BwdWs& w, bool dense, bool ste) {
  const int64_t T = a.T, d = a.d, F = a.F, r = a.r, Fp = pad64(F), ldv = vals_ld(F), ldm = meta_ld(F);
  static const uint8_t planning = 0;   // (sizes only: the pointers are not set yet)
  const uint8_t* sm = a.s_meta ? a.s_meta : &planning;
  WgradPlan p;
  p.add(a.Z, r, nullptr, 0, a.dy, r, d, a.dV_down, r, false);
  if (dense) p.add(a.s_vals, F, nullptr, 0, w.dZ, F, r, a.dU_down, F, false);
  else p.add(a.s_vals, ldv, sm, ldm, w.dZ, Fp, r, a.dU_down, F, false);
  if (dense || ste) p.add(w.dH, Fp, nullptr, 0, a.P_in, F, r, a.dV_up, F, true);
  else p.add(w.dH, ldv, sm, ldm, a.P_in, Fp, r, a.dV_up, F, true);
  p.add(a.x, d, nullptr, 0, w.dP, d, r, a.dU_up, d, false);
  p.finish(T);
  p.g.part = w.part;
  return p;
}
// dH is compressed [T x ldv] in the sparse backward and dense [T x F] in the
// dense and straight-through ones, at a pitch of whole cache lines (at d_ff = 2736 or
// 5464 a 64-feature piece of a row of F would straddle two; us, pitch F against Fp:
// 350M dense, 32768 tokens, dH 123 / 118, dP 62.5 / 59; 1B dense, 16384, 147 / 139,
// 105 / 94, weight gradients 244 / 231; straight-through 1B, 32768, 401 / 386, 169 /
// 165, 519 / 492).  The straight-through backward also holds V_up^T (relu(h) is
// recomputed tile by tile inside the dH kernel).
BwdWs bwd_ws(char* p, int64_t T, int64_t d, int64_t F, int64_t r, bool dense, bool ste) {
  const int64_t Fp = pad64(F);
  Carver c{p};
  BwdWs w{};
  w.dZ = c.take<uint16_t>(T * r);
  w.dH = c.take<uint16_t>(T * ((dense || ste) ? Fp : vals_ld(F)));
  w.dP = c.take<uint16_t>(T * r);
  if (ste) w.V_upT = c.take<uint16_t>(Fp * r);
  w.V_upB = c.take<uint16_t>(pad256(r) * Fp);
  w.V_downB = c.take<uint16_t>(pad256(r) * pad64(d));
  if (!ste && route_wide(T, F, r, dense, bwd_lays_out(T, d, F, r, dense, ste)) == RESIDENT) w.U_downR = c.take<uint16_t>(Fp * r);
  if (route_down(T, d, r) == RESIDENT) w.U_upR = c.take<uint16_t>(pad64(d) * r);
  // partials: the weight gradients', and split-K of the long-K bf16 products at
  // small token counts (b1, b5, b8)
  size_t pb = T > 0 ? wgrad_plan(FfnArgs{T, d, F, r}, w, dense, ste).part_floats() * sizeof(float) : 0;
  pb = std::max(pb, small_split_bytes(T, r, d, 64));
  pb = std::max(pb, small_split_bytes(T, r, Fp, 64));
  pb = std::max(pb, small_split_bytes(T, d, r, 64));
  w.part = c.take<float>(pb / sizeof(float));
  w.bytes = c.used;
  return w;
}

#define ELAS_TRY(...)                        \
  do {                                       \
    hipError_t e_ = (__VA_ARGS__);           \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

}  // namespace

size_t spmm_workspace_bytes(int64_t K, int64_t N, int b_layout) {
  return b_layout == 0 ? align_up((size_t)K * N * sizeof(uint16_t)) : 0;
}

size_t fwd_workspace_bytes(int64_t T, int64_t d, int64_t F, int64_t r, bool dense, bool ab, bool lean) {
  return fwd_ws(nullptr, T, d, F, r, dense, ab, lean).bytes;
}

size_t bwd_workspace_bytes(int64_t T, int64_t d, int64_t F, int64_t r, bool dense, bool ste) {
  return bwd_ws(nullptr, T, d, F, r, dense, ste).bytes;
}

hipError_t run_spmm24(const uint16_t* a_vals, const uint8_t* a_meta, int64_t M, int64_t K, const uint16_t* b,
                      int64_t N, bool b_is_nk, uint16_t* c, void* ws, hipStream_t st) {
  if (M == 0) return hipSuccess;
  const uint16_t* bt = b;
  int64_t ldb = K;
  if (!b_is_nk) {   // B [K x N] -> B^T [N x K] in the workspace
    uint16_t* t = (uint16_t*)ws;
    ELAS_TRY(transpose_pad(b, K, N, N, t, N, K, K, st));
    bt = t;
  }
  GemmArgs g{};
  g.A = a_vals; g.lda = vals_ld(K); g.Am = a_meta; g.ldam = meta_ld(K);
  g.B = bt; g.ldb = ldb;
  g.M = M; g.N = N; g.K = pad64(K); g.m_valid = M; g.ka_valid = pad64(K); g.kb_valid = K;
  g.C = c; g.ldc = N;
  return launch_sp("spmm24", g, st);
}

hipError_t run_fwd(const FfnArgs& a, hipStream_t st) {
  const int64_t T = a.T, d = a.d, F = a.F, r = a.r, Fp = pad64(F);
  const FwdWs w = fwd_ws((char*)a.ws, T, d, F, r, a.dense, a.ab, a.lean);
  // Weight factors K-contiguous for the MFMA operands: laid out here, or
  // given so (ELAS_FACTORS_AB: unpadded d_ff, whose missing rows / columns
  // the loads read as zero, exactly like the zero padding of the copies).
  const uint16_t *U_upT = a.U_up, *V_upT = a.V_up, *U_downT = a.U_down, *V_downT = a.V_down;
  int64_t F_rows = F, ld_ud = F;   // rows of V_up^T, pitch (= K extent) of U_down^T
  const bool fused = !a.dense && a.fused == 1;
  const Route up = fused ? TILED : fwd_up(T, F, r, a.dense, a.ab, a.lean), down = fused ? TILED : fwd_down(T, d, r, a.lean, a.ab, up);
  // The token-resident products take V_up^T and V_down^T in fragment order.
  const int64_t kp_up = up == RESIDENT ? r / 64 : 0, kp_down = down == RESIDENT ? r / 64 : 0;
  Transposes tr;
  if (!a.ab) {
    tr.add(a.U_up, d, r, r, w.U_upT, r, d, d);                                    // [r x d]
    tr.add(a.V_up, r, F, F, w.V_upT, Fp, r, r, 1, 0, kp_up);                      // [Fp x r], zero rows >= F
    tr.add(a.U_down, F, r, r, w.U_downT, r, Fp, Fp);                              // [r x Fp], zero cols >= F
    tr.add(a.V_down, r, d, d, w.V_downT, kp_down ? pad64(d) : d, r, r, 1, 0, kp_down);   // [d x r]
    U_upT = w.U_upT; V_upT = w.V_upT; U_downT = w.U_downT; V_downT = w.V_downT;
    F_rows = Fp;
    ld_ud = Fp;
  } else {
    if (kp_up) {
      tr.add(a.V_up, F, r, r, w.V_upT, Fp, r, r, 0, 0, kp_up);
      V_upT = w.V_upT;
    }
    if (kp_down) {
      tr.add(a.V_down, d, r, r, w.V_downT, pad64(d), r, r, 0, 0, kp_down);
      V_downT = w.V_downT;
    }
  }
  ELAS_TRY(tr.launch(st));
  // The one-launch forward only on request: measured slower than the four
  // kernels below at every supported shape but one.
  if (fused)
    return run_fused_fwd(a.x, U_upT, V_upT, U_downT, V_downT, T, d, F, r, F_rows, ld_ud, a.y, a.P, a.s_vals,
                         a.s_meta, a.Z, st);
  // P = x U_up
  if (route_long<false>(T, r, d) == SMALL)
    ELAS_TRY(launch_small_long<false>("k1_up_gemm", small_dense(U_upT, d, r, d, a.x, d, T, a.P), tiled_chunks(T, r, d), st));
  else
    ELAS_TRY(gemm_nt_bf16("k1_up_gemm", a.x, d, U_upT, d, a.P, r, T, r, d, st, w.part));
  ResArgs q{};   // the up projection
  q.W = V_upT; q.X = a.P; q.ldx = r; q.T = T; q.nfb = (int)(Fp / 64);
  if (!a.dense) {
    // H^T = V_up^T P^T with ReLU^2 + 2:4 selection + compression in the epilogue
    const char* tag = "k2_up_relu2_sparsify";
    q.sv = a.s_vals; q.sm = a.s_meta; q.ldv = vals_ld(F); q.ldm = meta_ld(F);
    if (up == SMALL) {
      SmallArgs g = small_dense(V_upT, r, F, r, a.P, r, T, nullptr);
      g.M = (int)Fp;
      g.sv = a.s_vals; g.sm = a.s_meta; g.ldv = vals_ld(F); g.ldm = meta_ld(F);
      ELAS_TRY(launch_small_short<EPI_SPARSIFY>(tag, g, st));
    } else if (up == RESIDENT) {
      ELAS_TRY(launch_resident<EPI_SPARSIFY>(tag, r, q, st));
    } else {
      GemmArgs g{};
      g.A = V_upT; g.lda = r; g.B = a.P; g.ldb = r;
      g.M = Fp; g.N = T; g.K = r; g.m_valid = F_rows; g.ka_valid = r; g.kb_valid = r;
      g.sv = a.s_vals; g.sm = a.s_meta; g.ldv = vals_ld(F); g.ldm = meta_ld(F); g.tok = T;   // S written tiled
      ELAS_TRY(launch_staged<EPI_SPARSIFY>(tag, g, st));
    }
    // Z = S U_down on the 2:4 operand
    if (route_long<true>(T, r, Fp) == SMALL) {
      ELAS_TRY(launch_small_long<true>("k3_spmm_down", small_sp(U_downT, ld_ud, r, F, a.s_vals, a.s_meta, T, a.Z), tiled_chunks(T, r, Fp), st));
    } else {
      GemmArgs z{};
      z.A = a.s_vals; z.lda = vals_ld(F); z.Am = a.s_meta; z.ldam = meta_ld(F); z.a_tiled = 1; z.tok = T;
      z.B = U_downT; z.ldb = ld_ud;
      z.M = T; z.N = r; z.K = Fp; z.m_valid = T; z.ka_valid = Fp; z.kb_valid = ld_ud;
      z.C = a.Z; z.ldc = r;
      ELAS_TRY(launch_sp("k3_spmm_down", z, st, w.part));
    }
  } else {
    // dense activations: S = relu(H)^2 written [T x F], then a dense product
    const char* tag = "k2_up_relu2_dense";
    q.C = a.s_vals; q.ldc = F; q.f_valid = (int)F;
    if (up == RESIDENT) {
      ELAS_TRY(launch_resident<EPI_ACT_DENSE>(tag, r, q, st));
    } else {
      ELAS_TRY(gemm_nt<EPI_ACT_DENSE>(tag, a.P, r, V_upT, r, a.s_vals, F, T, F, r, st));
    }
    if (route_long<false>(T, r, F) == SMALL)
      ELAS_TRY(launch_small_long<false>("k3_down_gemm_dense", small_dense(U_downT, ld_ud, r, F, a.s_vals, F, T, a.Z), tiled_chunks(T, r, F), st));
    else
      ELAS_TRY(gemm_nt_bf16("k3_down_gemm_dense", a.s_vals, F, U_downT, ld_ud, a.Z, r, T, r, F, st, w.part));
  }
  // Y = Z V_down
  if (down == SMALL) return launch_small_down("k4_down_gemm", small_dense(V_downT, r, d, r, a.Z, r, T, a.y), st);
  if (down == RESIDENT) return resident_bf16("k4_down_gemm", V_downT, a.Z, T, d, r, a.y, st);
  ELAS_TRY(gemm_nt_bf16("k4_down_gemm", a.Z, r, V_downT, r, a.y, d, T, d, r, st, w.part));
  return hipSuccess;
}

// Full-rank ReLU^2 FFN forward (the comparison of Table 3, Sec. 4.2.3).  The
// weights come in the orientation of Eq. 1 (W_up [F x d], W_down [d x F]),
// which is already the K-contiguous operand layout, so nothing is re-laid out:
// S = relu(x W_up^T)^2 with the activation in the product's epilogue, then
// Y = S W_down^T.
hipError_t run_fullrank_fwd(const uint16_t* x, const uint16_t* W_up, const uint16_t* W_down, int64_t T,
                            int64_t d, int64_t F, uint16_t* y, uint16_t* S, hipStream_t st) {
  ELAS_TRY(gemm_nt<EPI_ACT_DENSE>("fr_up_relu2", x, d, W_up, d, S, F, T, F, d, st));
  // Y = S W_down^T
  ELAS_TRY(gemm_nt_bf16("fr_down_gemm", S, F, W_down, F, y, d, T, d, F, st));
  return hipSuccess;
}

hipError_t run_bwd(const FfnArgs& a, hipStream_t st) {
  const int64_t T = a.T, d = a.d, F = a.F, r = a.r, Fp = pad64(F);
  const int64_t ldv = vals_ld(F), ldm = meta_ld(F);
  if (T == 0) {
    ELAS_TRY(fill_zero(a.dU_up, d * r, st));
    ELAS_TRY(fill_zero(a.dV_up, r * F, st));
    ELAS_TRY(fill_zero(a.dU_down, F * r, st));
    ELAS_TRY(fill_zero(a.dV_down, r * d, st));
    return hipSuccess;
  }
  const BwdWs w = bwd_ws((char*)a.ws, T, d, F, r, a.dense, a.ste);
  // V_up and V_down are the K-contiguous B operands of dP and dZ as they are,
  // but the row pitch of V_up (d_ff elements) need not be a multiple of 64
  // bytes, so that each 128-byte row piece of a K step would straddle two
  // cache lines.  Both are copied blocked (one contiguous 32 KB block per
  // tile K step: measured 7 % faster for dP at 1B), and V_up^T for the
  // straight-through backward, in one launch.
  const bool sp = !a.dense && !a.ste;   // dH compressed
  const Route rz = route_long<false>(T, r, d), rp = route_over_ff(T, F, r, sp), down = route_down(T, d, r);
  const Route wide = a.ste ? TILED : route_wide(T, F, r, a.dense, bwd_lays_out(T, d, F, r, a.dense, a.ste));
  const int64_t nsk_vu = Fp / 64, nsk_vd = pad64(d) / 64;
  {
    Transposes tr;
    if (rp == TILED) tr.add(a.V_up, r, F, F, w.V_upB, pad256(r), Fp, 0, 0, nsk_vu);
    if (rz == TILED) tr.add(a.V_down, r, d, d, w.V_downB, pad256(r), pad64(d), 0, 0, nsk_vd);
    if (a.ste) tr.add(a.V_up, r, F, F, w.V_upT, Fp, r, r);      // [Fp x r], zero rows >= F
    if (wide == RESIDENT) tr.add(a.U_down, F, r, r, w.U_downR, Fp, r, r, 0, 0, r / 64);
    if (down == RESIDENT) tr.add(a.U_up, d, r, r, w.U_upR, pad64(d), r, r, 0, 0, r / 64);
    ELAS_TRY(tr.launch(st));
  }
  // dZ = dY V_down^T
  if (rz == SMALL)
    ELAS_TRY(launch_small_long<false>("b1_dZ", small_dense(a.V_down, d, r, d, a.dy, d, T, w.dZ), tiled_chunks(T, r, d), st));
  else
    ELAS_TRY(gemm_nt_bf16("b1_dZ", a.dy, d, w.V_downB, d, w.dZ, r, T, r, d, st, w.part, nsk_vd));
  ResArgs q{};   // dS = dZ U_down^T
  q.W = w.U_downR; q.X = w.dZ; q.ldx = r; q.T = T; q.nfb = (int)(Fp / 64);
  if (sp) {
    // dH = (dZ U_down^T) * mask * 2 relu(H), computed as dS^T = U_down dZ^T
    const char* tag = "b3_dH_masked";
    q.sv = a.s_vals; q.sm = a.s_meta; q.ldv = ldv; q.ldm = ldm; q.dv = w.dH;
    if (wide == SMALL) {
      SmallArgs g = small_dense(a.U_down, r, F, r, w.dZ, r, T, nullptr);
      g.M = (int)Fp;
      g.sv = a.s_vals; g.sm = a.s_meta; g.ldv = ldv; g.ldm = ldm; g.dv = w.dH;
      ELAS_TRY(launch_small_short<EPI_DH>(tag, g, st));
    } else if (wide == RESIDENT) {
      ELAS_TRY(launch_resident<EPI_DH>(tag, r, q, st));
    } else {
      GemmArgs g{};
      g.A = a.U_down; g.lda = r; g.B = w.dZ; g.ldb = r;
      g.M = Fp; g.N = T; g.K = r; g.m_valid = F; g.ka_valid = r; g.kb_valid = r;
      g.sv = a.s_vals; g.sm = a.s_meta; g.ldv = ldv; g.ldm = ldm; g.dv = w.dH; g.tok = T;   // S read, dH written, tiled
      ELAS_TRY(launch_staged<EPI_DH>(tag, g, st));
    }
    // dP = dH V_up^T on the 2:4 operand (tiled kernel: V_up blocked)
    if (rp == SMALL) {
      ELAS_TRY(launch_small_long<true>("b5_spmm_dP", small_sp(a.V_up, F, r, F, w.dH, a.s_meta, T, w.dP), tiled_chunks(T, r, Fp), st));
    } else {
      GemmArgs p{};
      p.A = w.dH; p.lda = ldv; p.Am = a.s_meta; p.ldam = ldm; p.a_tiled = 1; p.tok = T;
      p.B = w.V_upB; p.ldb = 64; p.b_nsk = nsk_vu;
      p.M = T; p.N = r; p.K = Fp; p.m_valid = T; p.ka_valid = Fp; p.kb_valid = F;
      p.C = w.dP; p.ldc = r;
      ELAS_TRY(launch_sp("b5_spmm_dP", p, st, w.part));
    }
  } else {
    // dense dH [T x F] = dS * 2 r at every position: r = bf16(sqrt(s)) from the
    // dense S (dense mode), or relu(h) recomputed from P and V_up (straight-
    // through estimator of Eq. 4 after a sparse forward)
    GemmArgs g{};
    g.A = a.U_down; g.lda = r; g.B = w.dZ; g.ldb = r;
    g.M = Fp; g.N = T; g.K = r; g.m_valid = F; g.ka_valid = r; g.kb_valid = r;
    g.ld_act = F; g.ld_dact = Fp; g.f_valid = F; g.dact = w.dH;
    if (a.ste) {
      // one kernel per tile: h^T = V_up^T P^T over the first r contraction
      // steps (V_up^T rows >= F read as zero), relu(h) kept in registers, then
      // dS^T = U_down dZ^T over the next r
      g.A = w.V_upT; g.B = a.P_in; g.A2 = a.U_down; g.B2 = w.dZ;
      ELAS_TRY(launch_act<EPI_DH_STE>("b3_dH_ste", g, st));
    } else if (wide == RESIDENT) {
      q.C = w.dH; q.ldc = Fp; q.act = a.s_vals; q.ld_act = F; q.f_valid = (int)F;
      ELAS_TRY(launch_resident<EPI_DH_DENSE>("b3_dH_dense", r, q, st));
    } else {
      g.act = a.s_vals;
      ELAS_TRY(launch_act<EPI_DH_DENSE>("b3_dH_dense", g, st));
    }
    // dP = dH V_up^T (dense)
    if (rp == SMALL)
      ELAS_TRY(launch_small_long<false>("b5_dP_dense", small_dense(a.V_up, F, r, F, w.dH, Fp, T, w.dP), tiled_chunks(T, r, F), st));
    else
      ELAS_TRY(gemm_nt_bf16("b5_dP_dense", w.dH, Fp, w.V_upB, F, w.dP, r, T, r, F, st, w.part, nsk_vu));
  }
  // the four weight gradients
  ELAS_TRY(wgrad_plan(a, w, a.dense, a.ste).launch(a.dense ? "b2467_weight_grads_dense" : a.ste ? "b2467_weight_grads_ste"
                                                                                             : "b2467_weight_grads", st));
  // dx = dP U_up^T   (U_up [d x r] is already K-contiguous)
  if (down == SMALL) return launch_small_down("b8_dx", small_dense(a.U_up, r, d, r, w.dP, r, T, a.dx), st);
  if (down == RESIDENT) return resident_bf16("b8_dx", w.U_upR, w.dP, T, d, r, a.dx, st);
  ELAS_TRY(gemm_nt_bf16("b8_dx", w.dP, r, a.U_up, r, a.dx, d, T, d, r, st, w.part));
  return hipSuccess;
}

}  // namespace elas
