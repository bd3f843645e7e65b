// Batched complex GEMM on the gfx950 matrix cores.
//
//   C_b = alpha * op(A_b) * B_b + beta * C_b        (row-major, interleaved complex)
//
// FP64 (z64): every complex 16x16x4 tile product is four real
// v_mfma_f64_16x16x4_f64 products (Cr += Ar Br - Ai Bi, Ci += Ar Bi + Ai Br),
// i.e. 8 real flops per complex multiply-add, the count the roofline uses, or
// three in the three-product form.
// FP32 (c64): the same structure on v_mfma_f32_16x16x4_f32.
//
// Large outputs are cut into the tiles of gemm_tile.h, small ones go to k_gemm_ks
// below.  A launch covers batch x splits x tiles workgroups mapped XCD-contiguously.
#include "common.h"
#include "gemm_tile.h"
#include "kernels.h"
#include "mfma.h"

namespace feast {

namespace {

// Complex products take three real MFMAs per step (M3) in the single-problem
// complex64 kernels and in the FP64 trailing update and triangular solves.
// Other FP64 products and the plain grouped kernels keep four (the grouped
// trailing update has a three-product form of its own, k_gemm_grp_upd).
template <typename T> constexpr bool kM3 = sizeof(T) == 8;

// Waves per SIMD the register allocation must leave room for (512 registers a
// lane are shared by the waves of a SIMD).
template <typename T, int BN = kTileN> constexpr int kWaves = sizeof(T) == 8 && BN == kTileN ? 6 : 4;

template <typename T, int TA, bool SUB, int BN = kTileN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves<T, BN>)))
void k_gemm(const GemmArgs<T> d, int64_t grid_total) {
  gemm_tile<T, kTileM, BN, 2, TA, SUB ? kTileSub : kTileGen, kM3<T>>(
      d, xcd_remap(blockIdx.x, grid_total));
}

// Strides past the reach of a 32-bit offset, and C on A or on B's rows of another
// length (no wider than a tile, hence 64 columns): 64-bit addresses.
template <typename T, int TA, bool SUB>
__global__ __launch_bounds__(256)
void k_gemm_wide(const GemmArgs<T> d, int64_t grid_total) {
  gemm_tile<T, kTileM, 64, 2, TA, SUB ? kTileSub : kTileGen, kM3<T>, true>(
      d, xcd_remap(blockIdx.x, grid_total));
}

// The LU trailing update C -= A B: a name of its own, so that kernel traces and
// counters time that update alone.
template <typename T, int BM, int BN>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(BM == kTileM ? kWaves<T, BN> : (sizeof(T) == 8 ? 2 : 1))))
void k_gemm_update(const GemmArgs<T> d, int64_t grid_total) {
  gemm_tile<T, BM, BN, 2, 0, kTileSub, true>(d, xcd_remap(blockIdx.x, grid_total));
}

// C -= A B of the triangular solves (GEMM_SOLVE): three real products in FP64 too.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves<T>)))
void k_gemm_solve(const GemmArgs<T> d, int64_t grid_total) {
  gemm_tile<T, kTileM, kTileN, 2, 0, kTileSub, true>(d, xcd_remap(blockIdx.x, grid_total));
}

// The LU trailing update C -= A B on a fixed number of persistent workgroups, each
// filling one compute unit on its own: four tile groups of 256 threads and about 100 KB
// of LDS (in complex64 48 KB of it dynamic LDS that nothing reads), so that no
// second workgroup of any kernel fits beside it.  The compute units left over
// stay free for the next panel's factorisation on another stream.
// Workgroup w runs on XCD w mod 8; XCD x works through the tile range
// [x per, (x + 1) per) in rounds, NG consecutive tiles a workgroup per round.
constexpr int kPersistGroups = 4;

template <typename T>
__global__ __launch_bounds__(256 * kPersistGroups)
__attribute__((amdgpu_waves_per_eu(kPersistGroups)))
void k_gemm_upd_pers(const GemmArgs<T> d, int64_t total, int64_t per, int rounds) {
  constexpr int NG = kPersistGroups;
  const int64_t x = blockIdx.x & 7, j = blockIdx.x >> 3, p8 = gridDim.x >> 3;
  const int g = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 8));  // wave-uniform
  __shared__ uint32_t gcount[NG];
  if (threadIdx.x < NG) gcount[threadIdx.x] = 0;
  __syncthreads();
  uint32_t phase = 0;  // barriers this wavefront's group has passed, times 4
  for (int i = 0; i < rounds; ++i) {
    const int64_t lin = x * per + (i * p8 + j) * NG + g;
    const bool own = lin < total;
    gemm_tile<T, kTileM, kTileN, 2, 0, kTileSub, true, false, NG>(d, own ? lin : total - 1, own,
                                                                  &gcount[g], &phase);
  }
}

// C_b = C0_b - (shift[b] A2 - A) B_b (three-product form, as the trailing update).
template <typename T, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : kWaves<T>)))
void k_gemm_shift(const GemmArgs<T> d, int64_t grid_total) {
  gemm_tile<T, kTileM, kTileN, 2, 0, kTileShift, true, WIDE>(d, xcd_remap(blockIdx.x, grid_total));
}

// A group of independent problems in one launch: tab[e].tile0 is the first
// linear tile of problem e (increasing); a workgroup finds its problem by
// bisection over the table.
template <typename T>
__device__ inline int find_problem(const GemmArgs<T> *__restrict__ tab, int count, int64_t lin) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab[mid].tile0 <= lin) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <typename T, int TA, bool SUB, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : kWaves<T>)))
void k_gemm_grp(const GemmArgs<T> *__restrict__ tab, int count, int64_t grid_total) {
  const int64_t lin = xcd_remap(blockIdx.x, grid_total);
  const GemmArgs<T> d = tab[find_problem(tab, count, lin)];
  gemm_tile<T, kTileM, kTileN, 2, TA, SUB ? kTileSub : kTileGen, false, WIDE>(d, lin - d.tile0);
}

// The grouped LU trailing update C -= A B with three real products per complex
// step.  The batched form picks it (or the four-product loop) per precision and
// order from its tuned table.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves<T>)))
void k_gemm_grp_upd(const GemmArgs<T> *__restrict__ tab, int count, int64_t grid_total) {
  const int64_t lin = xcd_remap(blockIdx.x, grid_total);
  const GemmArgs<T> d = tab[find_problem(tab, count, lin)];
  gemm_tile<T, kTileM, kTileN, 2, 0, kTileSub, true>(d, lin - d.tile0);
}

// Products whose output is too small to fill the chip with 64 x 64 tiles (inner
// products U^* V of n x m blocks, n x m blocks times m x m or n x n matrices with a
// small m, the small calls): one workgroup per 16 FM x 16 FN output tile, its W
// wavefronts taking consecutive ranges of K and adding their sums in LDS in
// wavefront order (deterministic, no workspace, one launch).
//   bound: the latency of one wavefront's load -> MFMA chain, then the matrix
//   cores of the few compute units in use; operands go from global memory (or
//   L2) straight into the MFMA lane layout -- 16 consecutive columns of a row per
//   16 lanes, or 8 consecutive k per row of an untransposed A -- so that no
//   barrier stands between a load and its use, and the next step's loads are in
//   flight while the current one is multiplied.
// A lane holds k = 8 s + 2 (lane / 16) + {0, 1} of step s: the two MFMAs of a step
// take the even and the odd ones (any assignment of k to lanes is the same sum
// as long as A and B agree), and a row of A is read in 128-byte runs.
// Measured against the 64 x 64 tiles (complex128, us a call): 157 x 157 x 4001 of
// op = ^* 609 -> 40, 64 x 64 x 2003 307 -> 22, 2003 x 64 x 2003 308 -> 44,
// 200 x 30 x 200 35 -> 11, 4000 x 160 x 160 31 -> 26.
template <typename T, int TA, int FM, int FN, int W>
__global__ __launch_bounds__(64 * W) void k_gemm_ks(const GemmArgs<T> d, int64_t grid_total) {
  using Ops = mfma_ops<T>;
  using real = typename Ops::real;
  using acc_t = typename Ops::acc_t;
  __shared__ real red[W][8 * FM * FN][64];
  const int64_t tm = (d.M + 16 * FM - 1) / (16 * FM), tn = (d.N + 16 * FN - 1) / (16 * FN);
  int64_t lin = xcd_remap(blockIdx.x, grid_total);
  if (lin >= tm * tn * d.batch * d.splits) return;
  const int64_t tile = lin % (tm * tn);
  lin /= tm * tn;
  const int64_t bidx = lin % d.batch, split = lin / d.batch;
  const int64_t m0 = (tile / tn) * (16 * FM), n0 = (tile % tn) * (16 * FN);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int c16 = lane & 15, g = lane >> 4;
  // this workgroup's K range [8 t0, K) (kchunk is a multiple of 8 when split)
  const int64_t K = (split + 1) * d.kchunk < d.K ? (split + 1) * d.kchunk : d.K;
  const int64_t t0 = split * d.kchunk / 8, steps = (K + 7) / 8 - t0;
  const int64_t s0 = t0 + steps * w / W, s1 = t0 + steps * (w + 1) / W;

  // rows of C past M and columns past N read row M - 1 and column N - 1: their
  // sums are never stored
  const T *pa[FM], *pb[FN];
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int64_t r = m0 + 16 * a + c16, rc = r < d.M ? r : d.M - 1;
    pa[a] = d.A + bidx * d.sA + (TA == 0 ? rc * d.lda : rc);
  }
#pragma unroll
  for (int b = 0; b < FN; ++b) {
    const int64_t c = n0 + 16 * b + c16;
    pb[b] = d.B + bidx * d.sB + (c < d.N ? c : d.N - 1);
  }
  T ra[2][FM][2], rb[2][FN][2];
  auto load = [&](int64_t s, int o) {
    const int64_t k0 = 8 * s + 2 * g;
    if (8 * s + 8 <= K) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int a = 0; a < FM; ++a) ra[o][a][h] = pa[a][TA == 0 ? k0 + h : (k0 + h) * d.lda];
#pragma unroll
        for (int b = 0; b < FN; ++b) rb[o][b][h] = pb[b][(k0 + h) * d.ldb];
      }
    } else {  // the last, partial step: k past K read k = K - 1 and count as zero
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool in = k0 + h < K;
        const int64_t k = in ? k0 + h : K - 1;
#pragma unroll
        for (int a = 0; a < FM; ++a) {
          const T v = pa[a][TA == 0 ? k : k * d.lda];
          ra[o][a][h].x = in ? v.x : real(0);
          ra[o][a][h].y = in ? v.y : real(0);
        }
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          const T v = pb[b][k * d.ldb];
          rb[o][b][h].x = in ? v.x : real(0);
          rb[o][b][h].y = in ? v.y : real(0);
        }
      }
    }
  };
  acc_t cr[FM][FN], ci[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) cr[a][b][r] = ci[a][b][r] = 0;
  auto mul = [&](int o) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      real ar[FM], ai[FM];
#pragma unroll
      for (int a = 0; a < FM; ++a) {
        ar[a] = ra[o][a][h].x;
        ai[a] = TA == 0 ? ra[o][a][h].y : -ra[o][a][h].y;  // op(A) = A^*
      }
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          cr[a][b] = Ops::mma(ar[a], rb[o][b][h].x, cr[a][b]);
          ci[a][b] = Ops::mma(ar[a], rb[o][b][h].y, ci[a][b]);
        }
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          cr[a][b] = Ops::mma(-ai[a], rb[o][b][h].y, cr[a][b]);
          ci[a][b] = Ops::mma(ai[a], rb[o][b][h].x, ci[a][b]);
        }
    }
  };
  if (s0 < s1) load(s0, 0);
  for (int64_t s = s0; s < s1; s += 2) {  // two steps a turn: the buffer index is a constant
    if (s + 1 < s1) load(s + 1, 1);
    mul(0);
    if (s + 2 < s1) load(s + 2, 0);
    if (s + 1 < s1) mul(1);
  }

#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        red[w][2 * ((a * FN + b) * 4 + r)][lane] = cr[a][b][r];
        red[w][2 * ((a * FN + b) * 4 + r) + 1][lane] = ci[a][b][r];
      }
  __syncthreads();
  const real alr = static_cast<real>(d.alpha.x), ali = static_cast<real>(d.alpha.y);
  const real ber = static_cast<real>(d.beta.x), bei = static_cast<real>(d.beta.y);
  const bool use_beta = (ber != 0 || bei != 0);
  T *C = d.C + bidx * d.sC;
  T *P = (d.splits > 1) ? d.work + (split * d.batch + bidx) * d.M * d.N : nullptr;
  for (int q = w; q < 4 * FM * FN; q += W) {  // q = (tile, element of the lane)
    const int64_t row = m0 + 16 * (q / (4 * FN)) + Ops::out_row(lane, q & 3);
    const int64_t col = n0 + 16 * ((q >> 2) % FN) + c16;
    real xr = 0, xi = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      xr += red[v][2 * q][lane];
      xi += red[v][2 * q + 1][lane];
    }
    if (row < d.M && col < d.N) {
      T v;
      v.x = alr * xr - ali * xi;
      v.y = alr * xi + ali * xr;
      if (P) {
        P[row * d.N + col] = v;
        continue;
      }
      T *p = C + row * d.ldc + col;
      if (use_beta) {
        const T o = *p;
        v.x += ber * o.x - bei * o.y;
        v.y += ber * o.y + bei * o.x;
      }
      *p = v;
    }
  }
}

// Deterministic reduction of split-K partials: C = sum_s W_s + beta C.
template <typename T>
__global__ __launch_bounds__(256) void k_splitk_reduce(const GemmArgs<T> d) {
  const int64_t per = d.M * d.N;
  const int64_t idx = blockIdx.x * 256ll + threadIdx.x;
  if (idx >= per * d.batch) return;
  const int64_t b = idx / per, e = idx % per;
  const int64_t row = e / d.N, col = e % d.N;
  double sr = 0.0, si = 0.0;
  for (int s = 0; s < d.splits; ++s) {
    const T v = d.work[(s * d.batch + b) * per + e];
    sr += v.x;
    si += v.y;
  }
  T *C = d.C + b * d.sC + row * d.ldc + col;
  if (d.beta.x != 0.0 || d.beta.y != 0.0) {
    const T o = *C;
    sr += d.beta.x * o.x - d.beta.y * o.y;
    si += d.beta.x * o.y + d.beta.y * o.x;
  }
  T v;
  v.x = static_cast<decltype(v.x)>(sr);
  v.y = static_cast<decltype(v.y)>(si);
  *C = v;
}

// Workgroups of a launch over bm x bn tiles (a multiple of 8: xcd_remap).
template <typename T> int64_t padded_tiles(const GemmArgs<T> &d, int bm, int bn) {
  const int64_t total = ((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * d.batch * d.splits;
  return (total + 7) / 8 * 8;
}

// complex64 C -= A B takes 64 x 64 tiles unless padding N to their width costs more
// than they save: long launches on data with full mantissas run at the chip's power
// limit, where the wider tile's fewer LDS and operand reads per product count (3744 x
// 3744 x 256, 16 matrices: 148 -> 160 TFLOP/s; on data of few bits, below the limit,
// both 170; 160 columns on 192: 146 -> 130).  complex128: 80 and 81, the narrow one kept.
template <typename T> constexpr int kSubN = sizeof(T) == 8 ? 64 : kTileN;  // the wider one
template <typename T> int sub_tile_n(int64_t N) {
  const int64_t narrow = (N + kTileN - 1) / kTileN * kTileN, wide = (N + 63) / 64 * 64;
  return 15 * wide <= 16 * narrow ? kSubN<T> : kTileN;
}

// (each launch's grid is counted in the tiles of the kernel that it names)
template <typename T>
void launch_tiles(hipStream_t s, const GemmArgs<T> &d, int ta, int cfg) {
  // C -= op(A) B is recognised from alpha = -1, beta = 1 without split-K
  const bool sub = d.splits == 1 && d.alpha.x == -1.0 && d.alpha.y == 0.0 && d.beta.x == 1.0 &&
                   d.beta.y == 0.0;
  const bool tall = cfg == GEMM_UPDATE_TALL && ta == 0 && sub;
  // C on A, or on B with rows of another length: an output of at most 64 x 64 has one
  // workgroup (64 columns), which has read all its operands when it writes
  const bool wide = d.A == d.C || (d.B == d.C && (d.ldb != d.ldc || d.sB != d.sC)) ||
                    !tile_spans_fit(d, ta, tall ? 128 : kTileM);
  auto go = [&](auto kernel, int bm, int bn) {
    const int64_t padded = padded_tiles(d, bm, bn);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(padded)), dim3(256), 0, s, d, padded);
  };
  constexpr int M = kTileM, N = kTileN, NS = kSubN<T>;
  if (wide) {
    if (ta == 0)
      sub ? go(k_gemm_wide<T, 0, true>, M, 64) : go(k_gemm_wide<T, 0, false>, M, 64);
    else
      sub ? go(k_gemm_wide<T, 2, true>, M, 64) : go(k_gemm_wide<T, 2, false>, M, 64);
  } else if (ta == 0 && sub) {
    const bool narrow = sub_tile_n<T>(d.N) == N;
    if (tall)
      go(k_gemm_update<T, 128, 64>, 128, 64);
    else if (cfg == GEMM_SOLVE)
      go(k_gemm_solve<T>, M, N);
    else if (cfg == GEMM_UPDATE)
      narrow ? go(k_gemm_update<T, M, N>, M, N) : go(k_gemm_update<T, M, NS>, M, NS);
    else
      narrow ? go(k_gemm<T, 0, true>, M, N) : go(k_gemm<T, 0, true, NS>, M, NS);
  } else if (ta == 0) {
    go(k_gemm<T, 0, false>, M, N);
  } else {
    sub ? go(k_gemm<T, 2, true>, M, N) : go(k_gemm<T, 2, false>, M, N);
  }
}

template <typename T, int FM, int FN, int W>
void launch_ks(hipStream_t s, const GemmArgs<T> &d, int ta) {
  const int64_t total = ((d.M + 16 * FM - 1) / (16 * FM)) * ((d.N + 16 * FN - 1) / (16 * FN)) *
                        d.batch * d.splits;
  const int64_t padded = (total + 7) / 8 * 8;
  const dim3 grid(static_cast<unsigned>(padded));
  if (ta == 0)
    hipLaunchKernelGGL((k_gemm_ks<T, 0, FM, FN, W>), grid, dim3(64 * W), 0, s, d, padded);
  else
    hipLaunchKernelGGL((k_gemm_ks<T, 2, FM, FN, W>), grid, dim3(64 * W), 0, s, d, padded);
}

template <typename T> void launch_splitk_reduce(hipStream_t s, const GemmArgs<T> &d) {
  const int64_t n = d.M * d.N * d.batch;
  hipLaunchKernelGGL((k_splitk_reduce<T>), dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0,
                     s, d);
}

// Output tiles below which a product takes k_gemm_ks; from there on the tiles read less
// per flop and are as fast or faster.  complex128, us (k_gemm_ks, tiles):
//   op = 1: 448 tiles, K = 100 24, 20; 384, K = 364 50, 55; 400, K = 364 54, 54; 800,
//     K = 1500 322, 369; 960, K = 1500 407, 371
//   op = ^* (each K step reads other rows): 400, K = 100 21, 20; 800, K = 364 87, 101;
//     960, K = 1500 387, 406
// complex64, and complex128 with the tiles' three-product form: 400, K = 364 34, 28; 308,
// K = 364 25, 28.
template <typename T> int64_t small_tiles(int ta, int cfg, int64_t K) {
  if (ta != 0) return K > 128 ? 1024 : 512;
  const bool m3 = kM3<T> || cfg == GEMM_SOLVE || cfg == GEMM_UPDATE;
  return m3 || K < 512 ? 400 : K < 1024 ? 512 : 832;
}

// In-place products (C is A or B) need one workgroup per column block and keep the
// tiles.  In k_gemm_ks: sixteen wavefronts while that leaves units idle and the sum is
// long enough for them (157 x 157 x 4001, 100 tiles: 41 us against 46 with eight); four
// for a sum of up to 64; 32 x 16 tiles for many tiles, where the operands' traffic
// counts: eight wavefronts for a long sum (4000 x 160 x 4000: 349 us against 380), four
// for a short one, so that all workgroups fit at once (4000 x 160 x 160: 24 us against
// 26).
template <typename T>
void gemm_small(hipStream_t s, GemmArgs<T> d, int ta, int64_t work_elems) {
  const int64_t t16 = ((d.M + 15) / 16) * ((d.N + 15) / 16) * d.batch;
  // K ranges over several workgroups where the tiles leave compute units idle,
  // each range at least 512 long (32 k a wavefront), if the caller has a workspace
  if (d.work && t16 <= 128 && d.K >= 1024) {
    int64_t sp = std::min<int64_t>(256 / t16, d.K / 512);
    sp = std::min<int64_t>(sp, work_elems / (d.M * d.N * d.batch));
    if (sp > 1) {
      d.kchunk = ((d.K + sp - 1) / sp + 7) / 8 * 8;
      d.splits = static_cast<int32_t>((d.K + d.kchunk - 1) / d.kchunk);
    }
  }
  if (t16 <= 1024 && d.K <= 64)
    launch_ks<T, 1, 1, 4>(s, d, ta);
  else if (t16 * d.splits <= 256 && t16 <= 128)
    launch_ks<T, 1, 1, 16>(s, d, ta);
  else if (t16 > 1024 && d.K >= 1024)
    launch_ks<T, 2, 1, 8>(s, d, ta);
  else if (t16 > 1024)
    launch_ks<T, 2, 1, 4>(s, d, ta);
  else
    launch_ks<T, 1, 1, 8>(s, d, ta);
  if (d.splits > 1) launch_splitk_reduce<T>(s, d);
}

template <typename T>
void gemm_impl(hipStream_t s, GemmArgs<T> d, int ta, int cfg, int64_t work_elems) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0) return;
  if (d.K <= 0) {
    // C = beta C: a GEMM with an empty K range does exactly that.
    d.K = 0;
  }
  d.splits = 1;
  d.kchunk = d.K > 0 ? d.K : 1;
  const int64_t tiles =
      ((d.M + kTileM - 1) / kTileM) * ((d.N + kTileN - 1) / kTileN) * d.batch;
  // Long sums over one to four tiles a compute unit: four ranges of K, if the caller has
  // a workspace (complex128, us: 4000 x 160 x 4000, 315 tiles, 349 -> 318; 6000 x 60 x
  // 6000, 188 tiles, 337 -> 309; op = ^* and fewer tiles are no faster)
  const bool split = d.work && ta == 0 && d.K >= 2048 && tiles >= 160 && tiles < 1024 &&
                     4 * d.batch * d.M * d.N <= work_elems;
  if (d.A != d.C && d.B != d.C && cfg != GEMM_UPDATE_TALL && !split &&
      tiles < small_tiles<T>(ta, cfg, d.K))
    return gemm_small<T>(s, d, ta, work_elems);
  if (split) {
    d.kchunk = ((d.K + 3) / 4 + kTileK - 1) / kTileK * kTileK;
    d.splits = 4;
  }
  launch_tiles<T>(s, d, ta, ta == 0 ? cfg : static_cast<int>(GEMM_SQUARE));
  if (d.splits > 1) launch_splitk_reduce<T>(s, d);
}

}  // namespace

template <typename T>
GroupTiles gemm_group_tiles(GemmArgs<T> *tab, int count, int ta) {
  GroupTiles t{0, false};
  for (int e = 0; e < count; ++e) {
    tab[e].splits = 1;
    tab[e].kchunk = tab[e].K > 0 ? tab[e].K : 1;
    tab[e].tile0 = t.tiles;
    t.tiles += ((tab[e].M + kTileM - 1) / kTileM) * ((tab[e].N + kTileN - 1) / kTileN) * tab[e].batch;
    t.wide = t.wide || !tile_spans_fit(tab[e], ta, kTileM);
  }
  return t;
}
template GroupTiles gemm_group_tiles<z64>(GemmArgs<z64> *, int, int);
template GroupTiles gemm_group_tiles<c64>(GemmArgs<c64> *, int, int);

template <typename T>
void gemm_group(hipStream_t s, int ta, bool sub, const GemmArgs<T> *dtab, int count,
                GroupTiles t, int variant) {
  if (count <= 0 || t.tiles <= 0) return;
  const int64_t padded = (t.tiles + 7) / 8 * 8;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(padded)), dim3(256), 0, s, dtab, count,
                       padded);
  };
  if (ta != 0)
    t.wide ? go(k_gemm_grp<T, 2, false, true>) : go(k_gemm_grp<T, 2, false, false>);
  else if (!sub)
    t.wide ? go(k_gemm_grp<T, 0, false, true>) : go(k_gemm_grp<T, 0, false, false>);
  else if (t.wide)
    go(k_gemm_grp<T, 0, true, true>);
  else if (variant == GROUP_UPDATE_M3)
    go(k_gemm_grp_upd<T>);
  else
    go(k_gemm_grp<T, 0, true, false>);
}
template void gemm_group<z64>(hipStream_t, int, bool, const GemmArgs<z64> *, int, GroupTiles, int);
template void gemm_group<c64>(hipStream_t, int, bool, const GemmArgs<c64> *, int, GroupTiles, int);

void zgemm_shift_residual(hipStream_t s, int64_t M, int64_t N, int64_t K, const z64 *A,
                          const z64 *A2, int64_t lda, const z64 *shift, const z64 *Y, int64_t ldy,
                          int64_t sY, const z64 *R, int64_t ldr, int64_t sR, z64 *C, int64_t ldc,
                          int64_t sC, int32_t batch) {
  if (M <= 0 || N <= 0 || batch <= 0) return;
  GemmArgs<z64> d{M, N, K, A, lda, 0, Y, ldy, sY, C, ldc, sC, make_double2(-1.0, 0.0),
                  make_double2(1.0, 0.0), batch, 1, K > 0 ? K : 1, nullptr, 0, A2, shift, R, ldr, sR};
  const int64_t padded = padded_tiles(d, kTileM, kTileN);
  const dim3 grid(static_cast<unsigned>(padded));
  if (tile_spans_fit(d, 0, kTileM))
    hipLaunchKernelGGL((k_gemm_shift<z64, false>), grid, dim3(256), 0, s, d, padded);
  else
    hipLaunchKernelGGL((k_gemm_shift<z64, true>), grid, dim3(256), 0, s, d, padded);
}

template <typename T>
void update_persistent(hipStream_t s, GemmArgs<T> d, int wgs) {
  if (d.M <= 0 || d.N <= 0 || d.batch <= 0 || d.K <= 0) return;
  constexpr int NG = kPersistGroups;
  d.splits = 1;
  d.kchunk = d.K;
  const int64_t total = ((d.M + kTileM - 1) / kTileM) * ((d.N + kTileN - 1) / kTileN) * d.batch;
  // multiples of 8 (one share per XCD), no more than the tiles need
  int64_t p = std::max<int64_t>(8, wgs / 8 * 8);
  p = std::min<int64_t>(p, (total + 8 * NG - 1) / (8 * NG) * 8);
  const int64_t rounds = (total + p * NG - 1) / (p * NG);
  const int64_t per = rounds * (p / 8) * NG;
  hipLaunchKernelGGL((k_gemm_upd_pers<T>), dim3(static_cast<unsigned>(p)), dim3(256 * NG),
                     sizeof(T) == 8 ? 48 * 1024 : 0, s, d, total, per, static_cast<int>(rounds));
}

void zupdate_persistent(hipStream_t s, int64_t M, int64_t N, int64_t K, const z64 *A, int64_t lda,
                        int64_t sA, const z64 *B, int64_t ldb, int64_t sB, z64 *C, int64_t ldc,
                        int64_t sC, int32_t batch, int wgs) {
  GemmArgs<z64> d{M, N, K, A, lda, sA, B, ldb, sB, C, ldc, sC, make_double2(-1.0, 0.0),
                  make_double2(1.0, 0.0), batch, 1, K, nullptr, 0};
  update_persistent<z64>(s, d, wgs);
}

void cupdate_persistent(hipStream_t s, int64_t M, int64_t N, int64_t K, const c64 *A, int64_t lda,
                        int64_t sA, const c64 *B, int64_t ldb, int64_t sB, c64 *C, int64_t ldc,
                        int64_t sC, int32_t batch, int wgs) {
  GemmArgs<c64> d{M, N, K, A, lda, sA, B, ldb, sB, C, ldc, sC, make_double2(-1.0, 0.0),
                  make_double2(1.0, 0.0), batch, 1, K, nullptr, 0};
  update_persistent<c64>(s, d, wgs);
}

void zgemm(hipStream_t s, int transA, int64_t M, int64_t N, int64_t K, z64 alpha, const z64 *A,
           int64_t lda, int64_t sA, const z64 *B, int64_t ldb, int64_t sB, z64 beta, z64 *C,
           int64_t ldc, int64_t sC, int32_t batch, z64 *work, int64_t work_elems, int cfg) {
  GemmArgs<z64> d{M, N, K, A, lda, sA, B, ldb, sB, C, ldc, sC, alpha, beta, batch, 1, K, work, 0};
  gemm_impl<z64>(s, d, transA, cfg, work_elems);
}

void cgemm(hipStream_t s, int transA, int64_t M, int64_t N, int64_t K, z64 alpha, const c64 *A,
           int64_t lda, int64_t sA, const c64 *B, int64_t ldb, int64_t sB, z64 beta, c64 *C,
           int64_t ldc, int64_t sC, int32_t batch, c64 *work, int64_t work_elems, int cfg) {
  GemmArgs<c64> d{M, N, K, A, lda, sA, B, ldb, sB, C, ldc, sC, alpha, beta, batch, 1, K, work, 0};
  gemm_impl<c64>(s, d, transA, cfg, work_elems);
}

}  // namespace feast
