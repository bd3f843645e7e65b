// Triangular blocks of up to 64 rows in LDS, one workgroup of 256 threads (four
// wavefronts): solves and inverses by substitution in registers (wave_subst), and the
// pieces of the Gram blocks' Cholesky factor, whose inverse is built by halves
// ([L1 0; C L2]^-1 = [I1 0; -(I2 C) I1  I2]) with the products on the matrix cores.
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
// bk.. of the array)^*.  The two real products of each part are summed apart: their
// sums round at their own, smaller sizes (0.7 of the error of one sum of both).
template <typename T> struct Tile16 {
  using Ops = mfma_ops<T>;
  using real = typename Ops::real;
  typename Ops::acc_t rr, ii, ri, ir;
  __device__ Tile16() {
#pragma unroll
    for (int r = 0; r < 4; ++r) rr[r] = ii[r] = ri[r] = ir[r] = 0;
  }
  __device__ void step(T a, T b) {
    rr = Ops::mma(a.x, b.x, rr);
    ri = Ops::mma(a.x, b.y, ri);
    ii = Ops::mma(a.y, b.y, ii);
    ir = Ops::mma(a.y, b.x, ir);
  }
  __device__ real re(int r) const { return rr[r] - ii[r]; }
  __device__ real im(int r) const { return ri[r] + ir[r]; }
  template <bool CONJB>
  __device__ void mac(const T (*A)[kTP], int ai, int ak, const T (*B)[kTP], int bk, int bj, int ks,
                      int lane) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll 4
    for (int s = 0; s < ks; ++s) {
      const T a = A[ai + c][ak + 4 * s + g];
      T b = CONJB ? B[bj + c][bk + 4 * s + g] : B[bk + 4 * s + g][bj + c];
      if (CONJB) b.y = -b.y;
      step(a, b);
    }
  }
  // S[i0 + row][j0 + column] = sgn * tile
  __device__ void put(T (*S)[kTP], int i0, int j0, int lane, typename Ops::real sgn) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T v;
      v.x = sgn * re(r);
      v.y = sgn * im(r);
      S[i0 + Ops::out_row(lane, r)][j0 + (lane & 15)] = v;
    }
  }
};

// The values that lanes c, 16 + c, 32 + c and 48 + c hold, in each of the four.
template <typename T> __device__ inline void all_groups(T v, T (&o)[4]) {
  constexpr int N = sizeof(T) / 4;
  struct Words {
    uint32_t w[N];
  };
  const Words u = __builtin_bit_cast(Words, v);
  Words h[2], q[4];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const auto x = __builtin_amdgcn_permlane32_swap(u.w[i], u.w[i], false, false);
    h[0].w[i] = x[0];
    h[1].w[i] = x[1];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const auto x = __builtin_amdgcn_permlane16_swap(h[k].w[i], h[k].w[i], false, false);
      q[2 * k].w[i] = x[0];
      q[2 * k + 1].w[i] = x[1];
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = __builtin_bit_cast(T, q[k]);
}

// L x = b by substitution for 16 columns of right-hand sides, by one wavefront: L is
// the lower triangular matrix S, its rows of 16-row blocks k0 .. k1 - 1 (rows and
// columns before block k0 belong to entries of x that are zero).  Lane 16 g + c holds
// rows 4 q + g of column c from block k0 on: x[q] (q < 4 NB), zero past block k1.
// inv: reciprocals of the diagonal, where it does not count as ones (UNIT).  done(kb, x) gets
// block kb's four rows 16 kb + 4 p + g, p < 4.
// Four rows at a time: the four groups' entries go to all of them by swaps (no
// barrier), every group finishes the four rows for itself and takes them off its
// later rows of the block; the block then goes off the rows below on the matrix cores,
// whose operand and result layouts these are.  Only L's own entries are multiplied
// with: the product with an inverse that was built by halves had 1.6 times the error,
// and over- or underflowed for columns of very different size.
//   bound: the chain of 16 four-row steps a wavefront.
template <typename T, int NB, bool UNIT, typename Done>
__device__ __forceinline__ void wave_subst(const T (*S)[kTP], const T *inv, int k0, int k1,
                                           T (&x)[4 * NB], int lane, Done &&done) {
  const int c = lane & 15, g = lane >> 4;
  // the row of L whose sum the result element r of group g is: 4 r + g
  const int arow = sizeof(T) == 16 ? c : 4 * (c & 3) + (c >> 2);
  for (int kb = k0; kb < k1; ++kb) {
    const int o = 16 * kb;
    const T(*D)[kTP] = S + o;
    // L's entries within the four rows 4 q .. (the same in all lanes), read one step ahead
    T own[2][6], dia[2][4];
    auto fetch = [&](int q, int b) {
#pragma unroll
      for (int r = 0, e = 0; r < 4; ++r) {
#pragma unroll
        for (int k = 0; k < r; ++k, ++e) own[b][e] = D[4 * q + r][o + 4 * q + k];
        if constexpr (!UNIT) dia[b][r] = inv[o + 4 * q + r];
      }
    };
    fetch(0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      T v[4], low[3][4];  // (low: those of the later rows of the block)
#pragma unroll
      for (int p = q + 1; p < 4; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) low[p - 1][k] = D[4 * p + g][o + 4 * q + k];
      const int b = q & 1;
      if (q < 3) fetch(q + 1, b ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      all_groups(x[q], v);
#pragma unroll
      for (int r = 0, e = 0; r < 4; ++r) {
#pragma unroll
        for (int k = 0; k < r; ++k, ++e) v[r] = ffms(v[r], own[b][e], v[k]);
        if constexpr (!UNIT) v[r] = fmul(v[r], dia[b][r]);
      }
      x[q].x = g < 2 ? (g == 0 ? v[0].x : v[1].x) : (g == 2 ? v[2].x : v[3].x);
      x[q].y = g < 2 ? (g == 0 ? v[0].y : v[1].y) : (g == 2 ? v[2].y : v[3].y);
#pragma unroll
      for (int p = q + 1; p < 4; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) x[p] = ffms(x[p], low[p - 1][k], v[k]);
    }
    done(kb, x);
#pragma unroll
    for (int t = 1; t < NB; ++t)
      if (kb + t < k1) {
        Tile16<T> sum;
#pragma unroll
        for (int s = 0; s < 4; ++s) sum.step(D[16 * t + arow][o + 4 * s + g], x[s]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          x[4 * t + r].x -= sum.re(r);
          x[4 * t + r].y -= sum.im(r);
        }
      }
#pragma unroll
    for (int q = 0; q + 4 < 4 * NB; ++q) x[q] = x[q + 4];
  }
}

// Columns 16 w .. 16 w + 15 of the inverse of the lower triangular matrix S of nb blocks
// of 16 rows, by one wavefront (inv as in wave_subst): put(i, j, v) gets every entry of
// them that is not zero by position.
template <bool UNIT, typename T, typename Put>
__device__ __forceinline__ void wave_inverse64(const T (*S)[kTP], const T *inv, int nb, int lane,
                                               int w, Put &&put) {
  using Tr = cplx_traits<T>;
  const int c = lane & 15, g = lane >> 4, j = 16 * w + c;
  T x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = Tr::make(q < 4 && 4 * q + g == c ? 1.0 : 0.0, 0.0);
  wave_subst<T, 4, UNIT>(S, inv, w, nb, x, lane, [&](int kb, const T(&v)[16]) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int i = 16 * kb + 4 * p + g;
      if (i >= j) put(i, j, v[p]);
    }
  });
}

// In place: the inverse of the lower triangular 16 x 16 block at (o, o) of S, by one
// wavefront (two 8 x 8 blocks with one column per lane, then the 8 x 8 block between
// them).  Entries above the diagonal are not read and come out zero.
template <typename T> __device__ void wave_tri16(T (*S)[kTP], int o, int lane) {
  using Tr = cplx_traits<T>;
  {  // two 8 x 8 blocks, one column per lane (16 lanes' worth, repeated)
    const int d = o + (lane & 8), j = lane & 7;
    T x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = Tr::make(i == j ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = fmul(x[i], Tr::recip(S[d + i][d + i]));
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

}  // namespace feast
