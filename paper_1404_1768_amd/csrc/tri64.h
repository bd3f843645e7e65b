// Triangular 64 x 64 blocks in LDS: inverses by halves, the products on the
// matrix cores.  256 threads (four wavefronts) work on one block.
//
// A wavefront inverts a 16 x 16 diagonal block by itself (two 8 x 8 blocks with
// one column per lane, then the 8 x 8 off-diagonal block); four of them at once
// leave two levels of [L1 0; C L2]^-1 = [I1 0; -(I2 C) I1  I2] with 16 and 32 rows
// (I2 C first: the inverse X then has a small residual X L - I, the one that a
// solution X b inherits).
// The chain is 8 substitution steps and six products; a substitution over all 64
// rows with a barrier per row (one row published through LDS per step) takes 64
// steps of 0.6 us.
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"
#include "mfma.h"

namespace feast {

constexpr int kTP = 65;  // LDS row pitch: 16 rows of a 16-byte column fall on distinct banks

// Orders a wavefront's LDS accesses against later ones of its other lanes; the
// hardware runs one wavefront's LDS accesses in order, so only the compiler is held.
__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Complex products by fused multiply-adds.  a - b c rounds the product at its own size
// and the difference once (two FMAs on a's part instead round at a's size twice: errors
// of an LU of random matrices 1.17 times as large).
template <typename T> __device__ inline T fmul(T a, T b) {
  T r;
  r.x = fma(a.x, b.x, -(a.y * b.y));
  r.y = fma(a.x, b.y, a.y * b.x);
  return r;
}
template <typename T> __device__ inline T ffms(T a, T b, T c) {  // a - b c
  a.x -= fma(b.x, c.x, -(b.y * c.y));
  a.y -= fma(b.x, c.y, b.y * c.x);
  return a;
}

// 16 x 16 complex tile products from LDS: c += A B over 4 ks values of k, A at
// (ai, ak) and B at (bk, bj) of their arrays; CONJB: B = (rows bj.., columns
// bk.. of the array)^*.
template <typename T> struct Tile16 {
  using Ops = mfma_ops<T>;
  typename Ops::acc_t re, im;
  __device__ Tile16() {
#pragma unroll
    for (int r = 0; r < 4; ++r) re[r] = im[r] = 0;
  }
  template <bool CONJB>
  __device__ void mac(const T (*A)[kTP], int ai, int ak, const T (*B)[kTP], int bk, int bj, int ks,
                      int lane) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll 4
    for (int s = 0; s < ks; ++s) {
      const T a = A[ai + c][ak + 4 * s + g];
      T b = CONJB ? B[bj + c][bk + 4 * s + g] : B[bk + 4 * s + g][bj + c];
      if (CONJB) b.y = -b.y;
      re = Ops::mma(a.x, b.x, re);
      im = Ops::mma(a.x, b.y, im);
      re = Ops::mma(-a.y, b.y, re);
      im = Ops::mma(a.y, b.x, im);
    }
  }
  // S[i0 + row][j0 + column] = sgn * tile
  __device__ void put(T (*S)[kTP], int i0, int j0, int lane, typename Ops::real sgn) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T v;
      v.x = sgn * re[r];
      v.y = sgn * im[r];
      S[i0 + Ops::out_row(lane, r)][j0 + (lane & 15)] = v;
    }
  }
};

// In place: the inverse of the lower triangular 16 x 16 block at (o, o) of S, by
// one wavefront.  unit: the diagonal counts as ones (what is stored there is
// replaced).  Entries above the diagonal are not read and come out zero.
template <typename T> __device__ void wave_tri16(T (*S)[kTP], int o, bool unit, int lane) {
  using Tr = cplx_traits<T>;
  {  // two 8 x 8 blocks, one column per lane (16 lanes' worth, repeated)
    const int d = o + (lane & 8), j = lane & 7;
    T x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = Tr::make(i == j ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (!unit) x[i] = fmul(x[i], Tr::recip(S[d + i][d + i]));
#pragma unroll
      for (int r = i + 1; r < 8; ++r) x[r] = ffms(x[r], S[d + r][d + i], x[i]);
    }
    wave_lds_order();
    if (lane < 16)
#pragma unroll
      for (int i = 0; i < 8; ++i) S[d + i][d + j] = x[i];
    wave_lds_order();
  }
  const int i = lane >> 3, j = lane & 7;
  T p = Tr::make(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < 8; ++k) p = ffms(p, S[o + 8 + i][o + 8 + k], S[o + 8 + k][o + j]);  // -(I2 C)
  wave_lds_order();
  p.x = -p.x;
  p.y = -p.y;
  S[o + 8 + i][o + j] = p;
  S[o + i][o + 8 + j] = Tr::make(0.0, 0.0);
  wave_lds_order();
  T q = Tr::make(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < 8; ++k) q = ffms(q, S[o + 8 + i][o + k], S[o + k][o + j]);  // -(I2 C) I1
  wave_lds_order();
  S[o + 8 + i][o + j] = q;
  wave_lds_order();
}

// In place: [I1 0; C I2] -> [I1 0; -(I2 C) I1  I2] with diagonal blocks of H rows
// already inverted, for the 32 / H blocks of S; 256 threads, barriers inside.
template <typename T, int H> __device__ void tri_join(T (*S)[kTP], int lane, int wave) {
  constexpr int HT = H / 16, TILES = HT * HT;  // tiles of a C block
  const bool on = wave < TILES * (32 / H);
  const int o = 2 * H * (wave / TILES), ti = 16 * (wave % TILES / HT), tj = 16 * (wave % TILES % HT);
  Tile16<T> p;
  if (on)  // I2 C: columns k < ti + 16 of I2 only
    p.template mac<false>(S, o + H + ti, o + H, S, o + H, o + tj, (ti + 16) / 4, lane);
  __syncthreads();
  if (on) p.put(S, o + H + ti, o + tj, lane, -1);
  __syncthreads();
  Tile16<T> q;
  if (on)  // (-I2 C) I1: rows k >= tj of I1 only
    q.template mac<false>(S, o + H + ti, o + tj, S, o + tj, o + tj, (H - tj) / 4, lane);
  __syncthreads();
  if (on) q.put(S, o + H + ti, o + tj, lane, 1);
  __syncthreads();
}

// In place: the inverse of the lower triangular 64 x 64 matrix S (a barrier has
// passed since it was written; one has passed when this returns).  The strict
// upper triangle of the 16 x 16 diagonal blocks comes out zero; the blocks above
// the diagonal blocks are neither read nor written.
template <typename T> __device__ void tri64_inverse(T (*S)[kTP], bool unit, int lane, int wave) {
  wave_tri16(S, 16 * wave, unit, lane);
  __syncthreads();
  tri_join<T, 16>(S, lane, wave);
  tri_join<T, 32>(S, lane, wave);
}

}  // namespace feast
