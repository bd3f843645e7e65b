// Blocked LU with partial pivoting of the shifted matrices z_j B - A (the
// shifted systems of eq. 4-4, factored once and reused, Section 4.3).
// Row-major storage: a row swap moves contiguous memory, and a panel row is a
// contiguous run of the panel width.
//
// Kernels here are the latency-bound parts of the factorisation; the flops of
// the trailing and panel updates run in the MFMA GEMM (k_gemm.hip).
#include <climits>

#include "common.h"
#include "kernels.h"
#include "tri64.h"

namespace feast {

namespace {

template <typename T> __device__ inline T czero() {
  T z;
  z.x = 0;
  z.y = 0;
  return z;
}

// 32-bit lane exchange through DPP (VALU, no LDS round trip); lanes that the
// pattern gives no source read 0, the identity of the unsigned maxima below.
template <int CTRL> __device__ inline uint32_t dpp32(uint32_t v) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ inline uint64_t dpp64(uint64_t v) {
  return (static_cast<uint64_t>(dpp32<CTRL>(static_cast<uint32_t>(v >> 32))) << 32) |
         dpp32<CTRL>(static_cast<uint32_t>(v));
}
// Maximum of an unsigned key over the 64 lanes of a wavefront, returned
// uniformly: swaps inside quads, rotations inside rows of 16, then the
// broadcasts of lane 15 and lane 31 that leave the full maximum in lane 63.
__device__ inline uint64_t wave_max_u64(uint64_t k) {
  uint64_t o;
  o = dpp64<0xb1>(k);  // quad_perm [1,0,3,2]
  k = o > k ? o : k;
  o = dpp64<0x4e>(k);  // quad_perm [2,3,0,1]
  k = o > k ? o : k;
  o = dpp64<0x124>(k);  // row_ror:4
  k = o > k ? o : k;
  o = dpp64<0x128>(k);  // row_ror:8
  k = o > k ? o : k;
  o = dpp64<0x142>(k);  // row_bcast:15
  k = o > k ? o : k;
  o = dpp64<0x143>(k);  // row_bcast:31
  k = o > k ? o : k;
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(k), 63);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(k >> 32), 63);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Maximum over each row of 16 lanes, left in every lane of the row.
__device__ inline uint64_t row16_max_u64(uint64_t k) {
  uint64_t o;
  o = dpp64<0xb1>(k);
  k = o > k ? o : k;
  o = dpp64<0x4e>(k);
  k = o > k ? o : k;
  o = dpp64<0x124>(k);
  k = o > k ? o : k;
  o = dpp64<0x128>(k);
  k = o > k ? o : k;
  return k;
}
__device__ inline uint64_t uniform_u64(uint64_t k) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(k));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(k >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Pivot keys: |re| + |im| of a candidate as an unsigned integer that orders
// like the value (IEEE bits of a non-negative number, plus one so that 0 marks
// "no candidate"; NaN is no candidate).  complex64 packs the row index into
// the low half (complemented, so the lowest row wins a tie) and needs one
// reduction; complex128 breaks ties in a second reduction over the row index.
template <typename T> struct PivKey;
template <> struct PivKey<c64> {
  static constexpr bool kPacked = true;
  __device__ static uint64_t key(c64 a, int row) {
    const float v = fabsf(a.x) + fabsf(a.y);
    if (!(v >= 0.0f)) return 0;
    return (static_cast<uint64_t>(__float_as_uint(v)) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(row));
  }
};
template <> struct PivKey<z64> {
  static constexpr bool kPacked = false;
  __device__ static uint64_t key(z64 a, int) {
    const double v = fabs(a.x) + fabs(a.y);
    if (!(v >= 0.0)) return 0;
    return static_cast<uint64_t>(__double_as_longlong(v)) + 1;
  }
};

// Maxima of a key over the 64 lanes of a wavefront (returned uniformly) and over
// each row of 16 lanes (left in every lane of the row).  A lane that a pattern
// gives no source keeps its own value.  Keys are never NaN (v_max returns the
// other operand then) and -1 marks "no candidate".
template <int CTRL> __device__ inline float dpp_of(float x) {
  const int i = __float_as_int(x);
  return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ inline double dpp_of(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}
template <typename R> __device__ inline R row16_max(R x) {
  x = fmax(x, dpp_of<0xb1>(x));   // quad_perm [1,0,3,2]
  x = fmax(x, dpp_of<0x4e>(x));   // quad_perm [2,3,0,1]
  x = fmax(x, dpp_of<0x124>(x));  // row_ror:4
  return fmax(x, dpp_of<0x128>(x));  // row_ror:8
}
__device__ inline float lane_of(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ inline double lane_of(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}
template <typename R> __device__ inline R first_lane(R x) { return lane_of(x, 0); }
template <typename R> __device__ inline R wave_max(R x) {
  x = row16_max(x);
  x = fmax(x, dpp_of<0x142>(x));  // row_bcast:15
  x = fmax(x, dpp_of<0x143>(x));  // row_bcast:31: lane 63 holds the maximum
  return lane_of(x, 63);
}

// 1 / a for finite a != 0: a scaled by the power of two of its larger part, so
// that |a|^2 is in [1/4, 2), one real reciprocal (the hardware's estimate and
// Newton steps), a Newton step on the complex one, scaled back.  No intermediate
// overflows or underflows.
__device__ inline double rcp_newton(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}
__device__ inline float rcp_newton(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(r, fmaf(-d, r, 1.0f), r);
}
__device__ inline int exp_of(double x) { return __builtin_amdgcn_frexp_exp(x); }
__device__ inline int exp_of(float x) { return __builtin_amdgcn_frexp_expf(x); }
template <typename T> __device__ inline T recip_scaled(T a) {
  const int e = exp_of(fmax(fabs(a.x), fabs(a.y)));
  const auto x = ldexp(a.x, -e), y = ldexp(a.y, -e);
  const auto r = rcp_newton(fma(x, x, y * y));
  const auto u = x * r, v = -(y * r);
  const auto du = fma(y, v, fma(-x, u, decltype(r)(1))), dv = -fma(x, v, y * u);  // 1 - a o
  T o;
  o.x = ldexp(u + fma(u, du, -(v * dv)), -e);
  o.y = ldexp(v + fma(u, dv, v * du), -e);
  return o;
}

// One workgroup of NT threads per matrix holds the leaf columns [c0, c0+w)
// of rows [c0, n) in registers (thread t owns rows c0 + t + NT q) and factors
// them column by column with partial pivoting (largest |re|+|im|, lowest row
// on ties; Section 4.3 reuses these factors for every filter).
// Bound by latency: one chain per column -- key, DPP maximum over the wavefront
// (ballots find its row, so no second reduction for the index), post to LDS,
// one barrier, maximum over the posts, row exchange, rank-1 update by fused
// multiply-adds.  The winning lane posts its row and its pivot's reciprocal;
// posts are double-buffered by column parity, so one barrier per column
// suffices.  Loads and stores walk along rows and turn through LDS of the
// wavefront's own, without barriers.
// Measured (us a leaf of 8 columns with the solve of its rows, 16 matrices): complex128
// 200 rows 18.2, 1000 rows 23.2, 2000 rows 32.8; complex64 up to 1024 rows 15.2, up to
// 2048 20.6, 32 matrices of up to 4000 rows 29.1.  (With a reduction for the pivot's
// value and one for its row, and without the solve, the leaf took 18.3, 24.7, 30.7 and
// 16.7, 22.6, 33.0.)
template <typename T, int NT, int RPT, int IB>
__global__ __launch_bounds__(NT) void k_leaf(T *__restrict__ Mall, int64_t ld_in, int64_t stride,
                                             int64_t n_in, int64_t c0, int w, int64_t pk0,
                                             int pkb, int ue, int32_t *__restrict__ ipiv_all,
                                             int32_t *__restrict__ info_all,
                                             const GrpMat *__restrict__ grp, int nodes) {
  using Tr = cplx_traits<T>;
  using real = typename Tr::real;
  constexpr int NW = NT / 64;
  constexpr int SB = IB < 8 ? IB : 8, SG = IB / SB;  // staged columns, column groups
  static_assert(NW <= 16 && IB % SB == 0, "at most 16 wavefronts; whole column groups");
  const int b = blockIdx.x;
  const MatRef<T> mr = mat_of<T>(grp, nodes, Mall, ld_in, stride, n_in, b);
  T *M = mr.M;
  const int64_t ld = mr.ld, n = mr.n;
  if (c0 + w > n) return;  // (grouped: this matrix is already factored)
  int32_t *ipiv = ipiv_all + b * n_in;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ T stg_all[NW][64][SB + 1];
  __shared__ real s_key[2][16];
  __shared__ int s_row[2][16];
  __shared__ T s_inv[2][16];
  __shared__ T s_post[2][16][IB];
  __shared__ T s_crow[2][IB];
  __shared__ int s_pivs[IB];
  __shared__ T s_l[IB][IB];   // the leaf's rows (L11)
  int info_local = 0;
  // rows of this thread relative to c0: tid + NT q (32-bit: rows < 2^31)
  const int nrel = static_cast<int>(n - c0);

  // Each wavefront moves its own 64 rows of block q (SB consecutive lanes per row)
  // and turns them through LDS of its own into one row per lane: no barrier, and
  // every block's loads are in flight before the first is waited for (addresses
  // clamped into the matrix, a select instead of a branch).
  auto &stg = stg_all[wave];
  const int er = lane / SB, ec = lane % SB;  // this lane's row and column of 64 / SB rows
  const int row0 = 64 * wave + er;
  T *Mw = M + c0 * (ld + 1) + row0 * ld + ec;
  T a[RPT][IB];
#pragma unroll
  for (int q = 0; q < RPT; ++q)
#pragma unroll
    for (int h = 0; h < SG; ++h)
#pragma unroll
      for (int k = 0; k < SB; ++k) {
        const int dr = NT * q + (64 / SB) * k;
        a[q][SB * h + k] = Mw[(row0 + dr < nrel ? dr : -row0) * ld + (SB * h + ec < w ? SB * h : -ec)];
      }
#pragma unroll
  for (int q = 0; q < RPT; ++q)
#pragma unroll
    for (int h = 0; h < SG; ++h) {
#pragma unroll
      for (int k = 0; k < SB; ++k) {
        const bool in = row0 + NT * q + (64 / SB) * k < nrel && SB * h + ec < w;
        stg[er + (64 / SB) * k][ec] = in ? a[q][SB * h + k] : czero<T>();
      }
      wave_lds_order();
#pragma unroll
      for (int c = 0; c < SB; ++c) a[q][SB * h + c] = stg[lane][c];
      wave_lds_order();
    }

#pragma unroll
  for (int c = 0; c < IB; ++c) {
    if (c >= w) break;
    const int par = c & 1;
    // keys of this thread's candidates (relative rows c .. nrel-1; -1: none)
    real v[RPT];
    real best = -1;
    T cand = czero<T>();
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int r = tid + NT * q;
      const real k = fabs(a[q][c].x) + fabs(a[q][c].y);
      v[q] = (r >= c && r < nrel && k >= 0) ? k : real(-1);  // (NaN is no candidate)
      if (v[q] > best) {
        best = v[q];
        cand = a[q][c];
      }
    }
    const real wbest = wave_max(best);
    if (wbest >= 0) {
      // the lowest row holding the maximum: lowest q, then lowest lane (uniform)
      int wq = 0, wl = 0;
#pragma unroll
      for (int q = RPT - 1; q >= 0; --q) {
        const uint64_t hit = __builtin_amdgcn_ballot_w64(v[q] == wbest);
        if (hit) {
          wq = q;
          wl = static_cast<int>(__builtin_ctzll(hit));
        }
      }
#pragma unroll
      for (int q = 0; q < RPT; ++q)
        if (wq == q && lane == wl) {
#pragma unroll
          for (int k = 0; k < IB; ++k) s_post[par][wave][k] = a[q][k];
          // (cand is a[q][c]: an equal candidate of a lower q would have been hit)
          s_inv[par][wave] = recip_scaled(cand);
          s_key[par][wave] = wbest;
          s_row[par][wave] = tid + NT * q;
        }
    } else if (lane == 0) {
      s_key[par][wave] = -1;  // no candidate in this wavefront
    }
    if (tid == c)
#pragma unroll
      for (int k = 0; k < IB; ++k) s_crow[par][k] = a[0][k];
    __syncthreads();
    // the winner among the posts: lane v of every row of 16 reads post v
    const int pv = lane & 15;
    const real pk = pv < NW ? s_key[par][pv] : real(-1);
    const int prw = pv < NW ? s_row[par][pv] : 0;
    const real gk = first_lane(row16_max(pk));
    int prel = c;  // pivot row relative to c0
    T prow[IB];
    T inv = czero<T>();
    if (gk >= 0) {
      uint64_t hit = __builtin_amdgcn_ballot_w64(pk == gk) & 0xFFFF;
      int gw = static_cast<int>(__builtin_ctzll(hit));
      prel = __builtin_amdgcn_readlane(prw, gw);
      for (hit &= hit - 1; hit; hit &= hit - 1) {  // ties in value: the lowest row
        const int o = static_cast<int>(__builtin_ctzll(hit));
        const int orow = __builtin_amdgcn_readlane(prw, o);
        if (orow < prel) {
          prel = orow;
          gw = o;
        }
      }
#pragma unroll
      for (int k = 0; k < IB; ++k) prow[k] = s_post[par][gw][k];
      inv = s_inv[par][gw];
      if (!(gk < INFINITY)) inv = Tr::recip(prow[c]);
    } else {  // no comparable entry (NaN column): keep the diagonal row
#pragma unroll
      for (int k = 0; k < IB; ++k) prow[k] = s_crow[par][k];
      inv = Tr::recip(prow[c]);
    }
    if (gk == 0) inv = czero<T>();  // exact zero pivot
    if (!(gk > 0) && info_local == 0) info_local = static_cast<int>(c0) + c + 1;
    if (tid == 0) s_pivs[c] = static_cast<int>(c0) + prel;
    if (prel != c) {
      const int ptid = prel % NT, pq = prel / NT;
      if (tid == c)
#pragma unroll
        for (int k = 0; k < IB; ++k) a[0][k] = prow[k];
      if (wave == ptid / 64)
#pragma unroll
        for (int q = 0; q < RPT; ++q)
          if (q == pq && tid == ptid)
#pragma unroll
            for (int k = 0; k < IB; ++k) a[q][k] = s_crow[par][k];
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int r = tid + NT * q;
      if (r > c && r < nrel) {
        const T l = fmul(a[q][c], inv);
        a[q][c] = l;
#pragma unroll
        for (int k = c + 1; k < IB; ++k) a[q][k] = ffms(a[q][k], l, prow[k]);
      }
    }
  }

  if (ue > 0 && tid < IB)
#pragma unroll
    for (int c = 0; c < IB; ++c) s_l[tid][c] = a[0][c];
  __syncthreads();  // s_pivs, s_l
  if (tid < w) ipiv[c0 + tid] = s_pivs[tid];
  // The leaf's swaps (c0 + c <-> s_pivs[c], in order) applied to the other
  // columns of the panel as one gather.  Destinations: the w leaf rows and
  // each distinct pivot row below them; each thread finds the source of its
  // destination by walking the swaps backwards, and all sources are read
  // before any destination is written.
  // (two wavefronts walk one destination row's panel columns, so the walk is
  // wave-uniform)
  int pv_[IB];
#pragma unroll
  for (int c = 0; c < IB; ++c) pv_[c] = c < w ? __builtin_amdgcn_readfirstlane(s_pivs[c]) : -1;
  // panel columns (clipped to the matrix: in a grouped launch a wide panel can
  // extend past a smaller matrix's last column); the leaf's own columns are skipped
  const int ncol = static_cast<int>(pk0 + pkb <= n ? pkb : n - pk0);
  constexpr int H = (2 * IB * 128 + NT - 1) / NT;  // 2 w rows of pkb <= 128 columns
  const int64_t pcol = pk0 + (tid & 127);
  const bool pin = (tid & 127) < ncol && (pcol < c0 || pcol >= c0 + w);
  T v[H];
  int dst[H];  // destination row of slot h (uniform), -1: none
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int k = NT / 128 * h + (wave >> 1);
    v[h] = czero<T>();
    dst[h] = -1;
    if (k < 2 * w) {
      int key = -1;
      if (k < w) {
        key = static_cast<int>(c0) + k;
      } else {
        const int j = k - w;
        int pj = -1;
#pragma unroll
        for (int c = 0; c < IB; ++c)
          if (c == j) pj = pv_[c];
        bool first = pj >= c0 + w;
#pragma unroll
        for (int c = 0; c < IB; ++c)
          if (c < j && pv_[c] == pj) first = false;
        if (first) key = pj;
      }
      if (key >= 0) {
        int src = key;
#pragma unroll
        for (int c = IB - 1; c >= 0; --c)
          if (c < w) {
            const int top = static_cast<int>(c0) + c;
            if (src == top) src = pv_[c];
            else if (src == pv_[c]) src = top;
          }
        if (src != key || (ue > 0 && k < w)) {
          dst[h] = key;
          if (pin) v[h] = M[static_cast<int64_t>(src) * ld + pcol];
        }
      }
    }
  }
  // leaf columns back through the wavefront's LDS (row-contiguous stores)
#pragma unroll
  for (int q = 0; q < RPT; ++q)
#pragma unroll
    for (int h = 0; h < SG; ++h) {
#pragma unroll
      for (int c = 0; c < SB; ++c) stg[lane][c] = a[q][SB * h + c];
      wave_lds_order();
#pragma unroll
      for (int k = 0; k < SB; ++k) {
        const int dr = NT * q + (64 / SB) * k;
        if (row0 + dr < nrel && SB * h + ec < w) Mw[dr * ld + SB * h] = stg[er + (64 / SB) * k][ec];
      }
      wave_lds_order();
    }
  // the leaf's exchanged rows over the panel's columns, through the LDS of the
  // wavefronts that fetched them: row k's columns are with wavefronts
  // 2 (k mod NT / 128) and the next one, 64 each
  constexpr int RW = NT / 128;
  auto su = [&](int k, int col) -> T & {
    return (&stg_all[2 * (k % RW) + (col >> 6)][0][0])[(k / RW) * 64 + (col & 63)];
  };
  if (ue > 0)
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int k = RW * h + (wave >> 1);
      if (k < w) {
        su(k, tid & 127) = v[h];
        dst[h] = -1;  // (stored below)
      }
    }
  __syncthreads();  // every source of the exchanges has been read
#pragma unroll
  for (int h = 0; h < H; ++h)
    if (dst[h] >= 0 && pin) M[static_cast<int64_t>(dst[h]) * ld + pcol] = v[h];
  // the leaf's rows: U12 = L11^{-1} A12 in the columns up to ue, one column per
  // thread (the others only exchanged)
  if (ue > 0 && tid < 128 && pin) {
    T x[IB];
#pragma unroll
    for (int k = 0; k < IB; ++k) x[k] = k < w ? su(k, tid) : czero<T>();
    if (pcol >= c0 + w && pcol < c0 + w + ue)
#pragma unroll
      for (int k = 0; k < IB; ++k)
#pragma unroll
        for (int r = k + 1; r < IB; ++r)
          if (r < w) x[r] = ffms(x[r], s_l[r][k], x[k]);
#pragma unroll
    for (int k = 0; k < IB; ++k)
      if (k < w) M[(c0 + k) * ld + pcol] = x[k];
  }
  if (tid == 0 && info_local != 0 && info_all[b] == 0) info_all[b] = info_local;
}

// A panel's exchanges (rows r0 + i <-> ipiv[r0 + i], i < kb <= 128, in order) on
// the columns outside it, [0, clo) and [chi, n), as one gather: the exchanges
// reach at most the kb panel rows and kb rows below, and every destination's
// source is found by walking them backwards (all destinations at once, in LDS).
// A workgroup moves 512-byte pieces of those rows, every piece read before any is
// written.  One exchange after the other, each column waited for 128 memory round
// trips: 58 us a 128-column panel of 16 complex128 matrices of order 1000, 26 us
// so (124 us for 32 complex64 ones of order 4000, 95 to 107 so, 5 TB/s).
template <typename T>
__global__ __launch_bounds__(256) void k_laswp_outside(T *__restrict__ Mall, int64_t ld_in,
                                                       int64_t stride, int64_t n_in, int64_t r0,
                                                       int kb, int64_t clo, int64_t chi,
                                                       const int32_t *__restrict__ ipiv_all,
                                                       const GrpMat *__restrict__ grp, int nodes) {
  constexpr int CT = 512 / sizeof(T), G = 256 / CT;  // columns of a piece, rows at a time
  __shared__ int2 s_x[128];  // the exchanges that move rows: panel row, its partner
  __shared__ int s_dst[256], s_src[256];
  __shared__ int s_cnt[4];
  const int b = blockIdx.y;
  const MatRef<T> mr = mat_of<T>(grp, nodes, Mall, ld_in, stride, n_in, b);
  T *M = mr.M;
  const int64_t ld = mr.ld, n = mr.n;
  // (grouped: a panel wider than what is left of a smaller matrix is clipped
  // to its last row and column; a matrix already factored has nothing to swap)
  const int kbe = static_cast<int>(r0 + kb <= n ? kb : n - r0);
  const int64_t chie = chi < n ? chi : n, ncols = clo + (n - chie);
  if (kbe <= 0 || static_cast<int64_t>(blockIdx.x) * CT >= ncols) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // position of this thread among those with `on`, and their number
  auto rank_of = [&](bool on, int &count) {
    const uint64_t mask = __builtin_amdgcn_ballot_w64(on);
    if (lane == 0) s_cnt[wave] = __builtin_popcountll(mask);
    __syncthreads();
    int at = __builtin_popcountll(mask & ((1ull << lane) - 1));
    for (int w = 0; w < wave; ++w) at += s_cnt[w];
    count = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    __syncthreads();
    return at;
  };
  const int p = tid < kbe ? ipiv_all[b * n_in + r0 + tid] - static_cast<int>(r0) : tid;
  int nx, cnt;
  const int xat = rank_of(tid < kbe && p != tid, nx);
  if (nx == 0) return;
  if (tid < kbe && p != tid) s_x[xat] = make_int2(tid, p);
  __syncthreads();
  // destination (relative to r0): panel row tid, or the partner of exchange
  // tid - 128 if it lies below the panel and no earlier exchange names it
  int key = -1;
  if (tid < 128) key = tid < kbe ? tid : -1;
  else if (tid - 128 < nx && s_x[tid - 128].y >= kbe) key = s_x[tid - 128].y;
  int src = key, first = 0;  // first: the lowest exchange that names key
#pragma unroll 4
  for (int i = nx - 1; i >= 0; --i) {
    const int2 x = s_x[i];
    first = x.y == key ? i : first;
    src = src == x.x ? x.y : (src == x.y ? x.x : src);
  }
  const bool moved = key >= 0 && src != key && (tid < 128 || first == tid - 128);
  const int at = rank_of(moved, cnt);
  if (moved) {
    s_dst[at] = key;
    s_src[at] = src;
  }
  __syncthreads();
  const int g = tid / CT;
  for (int64_t c0 = static_cast<int64_t>(blockIdx.x) * CT; c0 < ncols;
       c0 += static_cast<int64_t>(gridDim.x) * CT) {
    const int64_t t = c0 + tid % CT;
    const bool in = t < ncols;
    T *C = M + r0 * ld + (!in ? 0 : t < clo ? t : chie + (t - clo));
    T v[CT];
#pragma unroll
    for (int e = 0; e < CT; ++e) {
      v[e] = czero<T>();
      if (in && G * e + g < cnt) v[e] = C[s_src[G * e + g] * ld];
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): every piece has arrived
    __syncthreads();
#pragma unroll
    for (int e = 0; e < CT; ++e)
      if (in && G * e + g < cnt) C[s_dst[G * e + g] * ld] = v[e];
  }
}

// Joins of the panel factorisation:
//   X = L11^{-1} X      for X = M[c0:c0+w1, c0+w1:c0+w1+w2], L11 unit lower (w1 x w1),
//   C -= L21 X          for C = M[c0+w1:n, c0+w1:c0+w1+w2], L21 = M[c0+w1:n, c0:c0+w1],
// in two launches: the small solve once per matrix (k_panel_solve, w1, w2 <= 64; a leaf
// that has solved its own rows needs none), then the update: for w1 <= 32 by every
// 64-row chunk and 32-column block (k_panel_rank, reading the solved X; bound by the
// traffic of C, so it runs on the VALU), else as a product.  (In one launch every
// chunk would repeat the solve.)
constexpr int kPU = 32;
// One workgroup per matrix, 16 columns of X per wavefront, by substitution (wave_subst).
//   64 x 64, 16 complex128 matrices: 12.2 us a launch (13.6 with products with inverted
//   16-row diagonal blocks, which left 1.6 times the residual).
template <typename T, int R>
__global__ __launch_bounds__(256) void k_panel_solve(T *__restrict__ Mall, int64_t ld_in,
                                                     int64_t stride, int64_t n_in, int64_t c0,
                                                     int w1, int w2,
                                                     const GrpMat *__restrict__ grp, int nodes) {
  __shared__ T sL[R][kTP];
  const MatRef<T> mr = mat_of<T>(grp, nodes, Mall, ld_in, stride, n_in, blockIdx.x);
  if (c0 + w1 + w2 > mr.n) return;
  const int64_t ld = mr.ld;
  T *D = mr.M + c0 * (ld + 1);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int PER = R / 4;  // rows of L11 a wavefront loads, rows of X a lane holds
  const int j = 16 * wave + (lane & 15);
  T v[PER], x[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = wave + 4 * k, r = 4 * k + g;
    v[k] = (i < w1 && lane < w1) ? D[i * ld + lane] : czero<T>();
    x[k] = (r < w1 && j < w2) ? D[r * ld + w1 + j] : czero<T>();
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) sL[wave + 4 * k][lane] = v[k];
  __syncthreads();
  if (16 * wave >= w2) return;
  wave_subst<T, R / 16, true>(sL, static_cast<const T *>(nullptr), 0, (w1 + 15) / 16, x, lane,
                        [&](int kb, const T(&y)[PER]) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int r = 16 * kb + 4 * p + g;
      if (r < w1 && j < w2) D[r * ld + w1 + j] = y[p];
    }
  });
}

template <typename T>
__global__ __launch_bounds__(256) void k_panel_rank(T *__restrict__ Mall, int64_t ld_in,
                                                    int64_t stride, int64_t n_in, int64_t c0,
                                                    int w1, int w2all,
                                                    const GrpMat *__restrict__ grp, int nodes) {
  using Tr = cplx_traits<T>;
  __shared__ T sL[64][kPU + 1];
  __shared__ T sX[kPU][kPU + 1];
  const MatRef<T> mr = mat_of<T>(grp, nodes, Mall, ld_in, stride, n_in, blockIdx.y);
  const int64_t ld = mr.ld, n = mr.n;
  if (c0 + w1 + w2all > n) return;
  T *M = mr.M + kPU * static_cast<int64_t>(blockIdx.z);  // (column block: M's columns past w1)
  const int w2 = w2all - kPU * static_cast<int>(blockIdx.z) < kPU ? w2all - kPU * static_cast<int>(blockIdx.z) : kPU;
  const T *L = mr.M;
  const int64_t r0 = c0 + w1 + static_cast<int64_t>(blockIdx.x) * 64;
  if (r0 >= n) return;  // (a chunk beyond a smaller matrix of a grouped launch)
  const int rows = static_cast<int>((n - r0 < 64) ? n - r0 : 64);
  const int tid = threadIdx.x;
  for (int e = tid; e < w1 * w2; e += 256) {
    const int i = e / w2, j = e % w2;
    sX[i][j] = M[(c0 + i) * ld + c0 + w1 + j];
  }
  for (int e = tid; e < rows * w1; e += 256) {
    const int i = e / w1, k = e % w1;
    sL[i][k] = L[(r0 + i) * ld + c0 + k];
  }
  const int ti = tid >> 4, tj = tid & 15;
  T c[4][2], acc[4][2];  // (the sum apart from C: it rounds at its own size)
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = ti + 16 * a, j = tj + 16 * b;
      acc[a][b] = Tr::make(0.0, 0.0);
      c[a][b] = (i < rows && j < w2) ? M[(r0 + i) * ld + c0 + w1 + j] : Tr::make(0.0, 0.0);
    }
  __syncthreads();
  for (int k = 0; k < w1; ++k) {
    T l[4], x[2];
#pragma unroll
    for (int a = 0; a < 4; ++a) l[a] = sL[ti + 16 * a][k];
#pragma unroll
    for (int b = 0; b < 2; ++b) x[b] = sX[k][tj + 16 * b];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        acc[a][b].x = fma(-l[a].y, x[b].y, fma(l[a].x, x[b].x, acc[a][b].x));
        acc[a][b].y = fma(l[a].y, x[b].x, fma(l[a].x, x[b].y, acc[a][b].y));
      }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = ti + 16 * a, j = tj + 16 * b;
      if (i >= rows || j >= w2) continue;
      c[a][b].x -= acc[a][b].x;
      c[a][b].y -= acc[a][b].y;
      M[(r0 + i) * ld + c0 + w1 + j] = c[a][b];
    }
}

// LU with partial pivoting (largest |re| + |im|, lowest row on ties, as the
// leaves) of small matrices held whole in LDS: a persistent grid whose
// workgroups take matrices b = blockIdx.x, blockIdx.x + gridDim.x, ... of a
// grouped table (order n_b <= NP), each factored column by column -- pivot
// search over the column, row exchange, multipliers, rank-1 update of the
// trailing block -- with the rows and columns spread over the 256 threads.
// Pivots (LAPACK order) to ipiv_all + b pstride, info_all[b] = 1 + the first
// column with an exact zero pivot (or 0).
template <typename T, int NP>
__global__ __launch_bounds__(256) void k_lu_small(const GrpMat *__restrict__ grp, int nodes,
                                                  int count, int64_t pstride,
                                                  int32_t *__restrict__ ipiv_all,
                                                  int32_t *__restrict__ info_all) {
  using Tr = cplx_traits<T>;
  using PK = PivKey<T>;
  static_assert(NP <= 256, "one row per thread in the pivot search");
  __shared__ T sM[NP][NP + 1];
  __shared__ T sl[NP];
  __shared__ uint64_t s_key[4];
  __shared__ int s_piv[NP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int b = blockIdx.x; b < count; b += gridDim.x) {
    const MatRef<T> mr = mat_of<T>(grp, nodes, static_cast<T *>(nullptr), 0, 0, 0, b);
    T *M = mr.M;
    const int64_t ld = mr.ld;
    const int n = static_cast<int>(mr.n);
    for (int e = tid; e < n * n; e += 256) {
      const int i = e / n, j = e - i * n;
      sM[i][j] = M[i * ld + j];
    }
    __syncthreads();
    int info = 0;
    for (int c = 0; c < n; ++c) {
      // pivot search: thread t looks at row c + t
      const int r = c + tid;
      uint64_t k = (r < n) ? PK::key(sM[r][c], r) : 0;
      uint64_t wk = wave_max_u64(k);
      if (lane == 0) s_key[wave] = wk;
      __syncthreads();
      uint64_t best = s_key[0];
      for (int w = 1; w < 4; ++w) best = s_key[w] > best ? s_key[w] : best;
      int p = c;
      if constexpr (PK::kPacked) {
        if (best != 0) p = static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(best));
      } else if (best != 0) {
        // ties in value: the lowest row among the candidates holding the maximum
        __syncthreads();
        const uint64_t ik = (k == best && k != 0) ? 0xFFFFFFFFull - static_cast<uint32_t>(r) : 0;
        wk = wave_max_u64(ik);
        if (lane == 0) s_key[wave] = wk;
        __syncthreads();
        uint64_t bi = s_key[0];
        for (int w = 1; w < 4; ++w) bi = s_key[w] > bi ? s_key[w] : bi;
        p = static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(bi));
      }
      if (best == 0 && info == 0) info = c + 1;  // (no comparable entry: keep the diagonal row)
      if (tid == 0) s_piv[c] = p;
      // exchange rows c and p
      if (p != c)
        for (int j = tid; j < n; j += 256) {
          const T x = sM[c][j];
          sM[c][j] = sM[p][j];
          sM[p][j] = x;
        }
      __syncthreads();
      const T piv = sM[c][c];
      const bool zero = piv.x == 0 && piv.y == 0;
      if (zero && info == 0) info = c + 1;
      const T inv = zero ? czero<T>() : Tr::recip(piv);
      if (r > c && r < n) {
        const T l = Tr::mul(sM[r][c], inv);
        sl[r] = l;
        sM[r][c] = l;
      }
      __syncthreads();
      // rank-1 update of the trailing block: thread (tr, tc) = (tid / 16, tid % 16)
      for (int i = c + 1 + (tid >> 4); i < n; i += 16) {
        const T l = sl[i];
        for (int j = c + 1 + (tid & 15); j < n; j += 16) sM[i][j] = Tr::fms(sM[i][j], l, sM[c][j]);
      }
      __syncthreads();
    }
    for (int e = tid; e < n * n; e += 256) {
      const int i = e / n, j = e - i * n;
      M[i * ld + j] = sM[i][j];
    }
    for (int i = tid; i < n; i += 256) ipiv_all[b * pstride + i] = s_piv[i];
    if (tid == 0) info_all[b] = info;
    __syncthreads();  // (sM, s_piv reused by the next matrix)
  }
}

// Inverse of one 64 x 64 diagonal block of each matrix (lower unit or upper
// non-unit), zero padded at out + b out_stride + I 64^2.  An upper block is
// inverted as the lower one it is with rows and columns in reverse order; a last
// block is worked in the 16-row pieces that it has, filled up with the identity.
// us a launch, complex128, by a substitution with a barrier per row, as an inverse put
// together from halves (whose products left twice the residual), and so: one 64-row
// block of 16 matrices 42, 12, 13; both triangles of 1024 matrices of order 64 71 (halves),
// 79 so; of 4096 matrices of order 8 218, 108.
template <typename T>
__global__ __launch_bounds__(256) void k_diag_inv(const T *__restrict__ Mall, int64_t ld_in,
                                                  int64_t stride, int64_t n_in, int64_t blk0,
                                                  bool lower_in, T *__restrict__ out_in,
                                                  T *__restrict__ other, int64_t out_stride,
                                                  const GrpMat *__restrict__ grp, int nodes) {
  __shared__ T S[64][kTP];
  __shared__ T s_inv[64];
  const bool lower = blockIdx.z == 0 ? lower_in : !lower_in;  // (z = 1: the other triangle)
  T *out = blockIdx.z == 0 ? out_in : other;
  const int64_t I = blk0 + blockIdx.x;
  const int b = blockIdx.y;
  const MatRef<const T> mr = mat_of<const T>(grp, nodes, Mall, ld_in, stride, n_in, b);
  const int64_t ld = mr.ld, r0 = I * 64;
  const int rb = static_cast<int>((mr.n - r0 < 64) ? mr.n - r0 : 64);  // (<= 0: past a smaller matrix)
  const T *D = mr.M + r0 * (ld + 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  T *o = out + b * out_stride + I * 4096;
  const int nb = rb > 0 ? (rb + 15) / 16 : 0, last = 16 * nb - 1;  // 16-row blocks of the matrix
  T v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int i = wave + 4 * k;
    const bool in = i < rb && lane < rb;
    v[k] = in ? D[i * ld + lane] : cplx_traits<T>::make(i == lane ? 1.0 : 0.0, 0.0);
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int i = wave + 4 * k;
    if (lower) S[i][lane] = v[k];
    else if (i <= last && lane <= last) S[last - i][last - lane] = v[k];
  }
  __syncthreads();
  if (!lower) {
    if (tid <= last) s_inv[tid] = cplx_traits<T>::recip(S[tid][tid]);
    __syncthreads();
  }
  // what the columns do not reach: the other triangle, and past the matrix
  for (int i = wave; i < 64; i += 4)
    if (i >= rb || lane >= rb || (lower ? lane > i : lane < i)) o[i * 64 + lane] = czero<T>();
  // (column block w costs nb - w steps: every other workgroup gives them to its
  // wavefronts in reverse order, so that a SIMD with one of each has its share)
  const int w = ((blockIdx.y ^ (blockIdx.y >> 8)) & 1) ? nb - 1 - wave : wave;
  if (w >= 0 && w < nb) {
    if (lower)
      wave_inverse64<true>(S, s_inv, nb, lane, w, [&](int i, int j, T x) {
        if (i < rb) o[i * 64 + j] = x;
      });
    else
      wave_inverse64<false>(S, s_inv, nb, lane, w, [&](int i, int j, T x) {
        if (last - j < rb) o[(last - i) * 64 + last - j] = x;
      });
  }
}

// Inverse of a 128-row diagonal block of a triangular factor from the inverses
// I1, I2 of its two 64-row halves (zero padded past the order) and the
// off-diagonal 64 x 64 block C of the factor:
//   lower (unit):  [L11 0; C L22]^{-1} = [I1 0; -I2 (C I1)  I2]
//   upper:         [U11 C; 0 U22]^{-1} = [I1  -(I1 C) I2; 0 I2]
// One workgroup per (block, matrix, triangle); the two 64 x 64 x 64 products run on the
// matrix cores from LDS, one 16-row strip of the output per wavefront.  (16
// complex128 matrices of order 200: 94 us a triangle with each thread summing its
// entries from LDS, 38 us for both so.)
template <typename T>
__global__ __launch_bounds__(256) void k_inv_pair(const T *__restrict__ F, int64_t ld,
                                                  int64_t fstride, int64_t n,
                                                  const T *__restrict__ Linv,
                                                  const T *__restrict__ Uinv, int64_t istride,
                                                  T *__restrict__ Linv2, T *__restrict__ Uinv2,
                                                  int64_t istride2) {
  const bool lower = blockIdx.z == 0;
  const T *inv64 = lower ? Linv : Uinv;
  T *inv128 = lower ? Linv2 : Uinv2;
  __shared__ T sA[64][kTP];
  __shared__ T sB[64][kTP];
  const int64_t B = blockIdx.x, b = blockIdx.y;
  const int64_t r0 = 128 * B;
  const int h2 = static_cast<int>((n - r0 - 64 < 64) ? n - r0 - 64 : 64);  // rows of the second half
  const T *M = F + b * fstride;
  const T *I1 = inv64 + b * istride + (2 * B) * 4096;
  const T *I2 = I1 + 4096;
  T *out = inv128 + b * istride2 + B * 16384;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the diagonal halves (the second one absent when h2 <= 0) and the zero block
  for (int i = wave; i < 64; i += 4) {
    const T d1 = I1[i * 64 + lane], d2 = h2 > 0 ? I2[i * 64 + lane] : czero<T>();
    out[i * 128 + lane] = d1;
    out[(64 + i) * 128 + 64 + lane] = d2;
    if (lower) out[i * 128 + 64 + lane] = czero<T>();
    else out[(64 + i) * 128 + lane] = czero<T>();
    // first product: lower C I1 (C = rows [r0+64, r0+64+h2) x cols [r0, r0+64)),
    //                upper I1 C (C = rows [r0, r0+64) x cols [r0+64, r0+64+h2))
    (lower ? sB : sA)[i][lane] = d1;
    if (lower) sA[i][lane] = i < h2 ? M[(r0 + 64 + i) * ld + r0 + lane] : czero<T>();
    else sB[i][lane] = lane < h2 ? M[(r0 + i) * ld + r0 + 64 + lane] : czero<T>();
    if (h2 <= 0) {
      if (lower) out[(64 + i) * 128 + lane] = czero<T>();
      else out[i * 128 + 64 + lane] = czero<T>();
    }
  }
  if (h2 <= 0) return;
  __syncthreads();
  Tile16<T> t[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) t[c].template mac<false>(sA, 16 * wave, 0, sB, 0, 16 * c, 16, lane);
  __syncthreads();
  // second product with the negated first one: lower I2 (-C I1), upper (-I1 C) I2
#pragma unroll
  for (int c = 0; c < 4; ++c) t[c].put(lower ? sB : sA, 16 * wave, 16 * c, lane, -1);
  for (int i = wave; i < 64; i += 4) (lower ? sA : sB)[i][lane] = I2[i * 64 + lane];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Tile16<T> x;
    x.template mac<false>(sA, 16 * wave, 0, sB, 0, 16 * c, 16, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * wave + mfma_ops<T>::out_row(lane, r), j = 16 * c + (lane & 15);
      T v;
      v.x = x.re(r);
      v.y = x.im(r);
      if (lower) out[(64 + i) * 128 + j] = v;
      else out[i * 128 + 64 + j] = v;
    }
  }
}

// n: order (pivot vectors of the batch are n_stride apart; grouped batches read
// each matrix's order from grp).
// Bound by latency: one exchange after the other costs an LDS round trip each.  So
// every wavefront takes 64 exchanges and follows, in registers, the 64 positions i and
// the 64 positions ipiv[i] back through them to where their entries come from (which
// depends on no entry); only moving the entries goes one wavefront after the other.
// n = 1000: 53 -> 8.6 us.
__global__ __launch_bounds__(1024) void k_perm(const int32_t *__restrict__ ipiv_all,
                                               int32_t *__restrict__ perm_all, int64_t n_stride,
                                               const GrpMat *__restrict__ grp, int nodes) {
  extern __shared__ int32_t sp[];
  const int b = blockIdx.x;
  const int n = static_cast<int>(grp ? grp[b / nodes].n : n_stride);
  const int32_t *ipiv = ipiv_all + b * n_stride;
  int32_t *perm = perm_all + b * n_stride;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < n; i += 1024) sp[i] = i;
  for (int k0 = 0; k0 < n; k0 += 1024) {
    const int i0 = k0 + 64 * wave, i = i0 + lane;
    const int p = i < n ? ipiv[i] : i;
    int a = i, c = p;
    if (i0 < n) {
#pragma unroll
      for (int j = 63; j >= 0; --j) {
        const int pj = __builtin_amdgcn_readlane(p, j), ij = i0 + j;
        a = a == ij ? pj : a == pj ? ij : a;
        c = c == ij ? pj : c == pj ? ij : c;
      }
    }
    for (int w = 0; w < 16 && k0 + 64 * w < n; ++w) {
      __syncthreads();
      if (wave == w && i < n) {
        const int32_t x = sp[a], y = sp[c];
        wave_lds_order();  // every lane's entries are read before any is written
        sp[i] = x;
        sp[p] = y;  // (lanes with the same p write the same entry)
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 1024) perm[i] = sp[i];
}

__global__ void k_fill_i32(int32_t *p, int64_t count, int32_t v) {
  const int64_t i = blockIdx.x * 256ll + threadIdx.x;
  if (i < count) p[i] = v;
}

template <typename T, int RPT, int IB, int NT = 1024>
void launch_leaf(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                 int64_t c0, int w, int64_t pk0, int pkb, int ue, int32_t *ipiv, int32_t *info,
                 const GrpMat *grp, int nodes) {
  hipLaunchKernelGGL((k_leaf<T, NT, RPT, IB>), dim3(batch), dim3(NT), 0, s, M, ld, stride, n, c0, w,
                     pk0, pkb, ue, ipiv, info, grp, nodes);
}

}  // namespace

template <> int leaf_max_width<z64>(int64_t rows) {
  if (rows <= 2048) return 8;
  if (rows <= 4096) return 4;
  if (rows <= 8192) return 2;
  if (rows <= 16384) return 1;
  return 0;
}
template <> int leaf_max_width<c64>(int64_t rows) {
  if (rows <= 4096) return 8;
  if (rows <= 8192) return 4;
  if (rows <= 16384) return 2;
  return 0;
}

template <>
bool leaf_lu<z64>(hipStream_t s, z64 *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                  int64_t c0, int w, int64_t pk0, int pkb, int ue, int32_t *ipiv, int32_t *info,
                  const GrpMat *grp, int nodes) {
  const int64_t rows = n - c0;
  if (w < 1 || w > leaf_max_width<z64>(rows) || pkb > 128) return false;
  // 256 threads up to 256 rows, where there may be many matrices (factorisations of 4096
  // of order 8: 224 us, 254 with 512 threads; of 400 of order 200 1335 and 1350; of 16 of
  // order 200 715 and 670); else 512: a leaf of 16 matrices of 1000 rows takes 23.2 us,
  // 26.2 with 256 threads and 24.5 with 1024; of 2000 rows 32.8, 31.2 with 1024, the
  // factorisation the same.
  if (rows <= 256)
    launch_leaf<z64, 1, 8, 256>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 512)
    launch_leaf<z64, 1, 8, 512>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 1024)
    launch_leaf<z64, 2, 8, 512>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 2048)
    launch_leaf<z64, 4, 8, 512>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 4096)
    launch_leaf<z64, 4, 4>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 8192)
    launch_leaf<z64, 8, 2>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else
    launch_leaf<z64, 16, 1>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  return true;
}

template <>
bool leaf_lu<c64>(hipStream_t s, c64 *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                  int64_t c0, int w, int64_t pk0, int pkb, int ue, int32_t *ipiv, int32_t *info,
                  const GrpMat *grp, int nodes) {
  const int64_t rows = n - c0;
  if (w < 1 || w > leaf_max_width<c64>(rows) || pkb > 128) return false;
  if (rows <= 1024)
    launch_leaf<c64, 1, 8>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 2048)
    launch_leaf<c64, 2, 8>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 4096)
    launch_leaf<c64, 4, 8>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else if (rows <= 8192)
    launch_leaf<c64, 8, 4>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  else
    launch_leaf<c64, 16, 2>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, ue, ipiv, info, grp, nodes);
  return true;
}

template <typename T>
void laswp_outside(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                   int64_t r0, int kb, int64_t clo, int64_t chi, const int32_t *ipiv,
                   const GrpMat *grp, int nodes) {
  // (n: the largest order of a grouped launch; every matrix has at most this many columns)
  const int64_t ncols = clo + (n > chi ? n - chi : 0);
  if (ncols <= 0 || kb <= 0) return;
  // one piece a workgroup while the chip has room for all, else several: finding
  // the sources costs a workgroup about as much as a piece
  constexpr int64_t ct = 512 / sizeof(T);
  const int64_t pieces = std::min<int64_t>((ncols + ct - 1) / ct, std::max<int64_t>(1, 1024 / batch));
  hipLaunchKernelGGL((k_laswp_outside<T>), dim3(static_cast<unsigned>(pieces), batch),
                     dim3(256), 0, s, M, ld, stride, n, r0, kb, clo, chi, ipiv, grp, nodes);
}
template void laswp_outside<z64>(hipStream_t, z64 *, int64_t, int64_t, int32_t, int64_t, int64_t,
                                 int, int64_t, int64_t, const int32_t *, const GrpMat *, int);
template void laswp_outside<c64>(hipStream_t, c64 *, int64_t, int64_t, int32_t, int64_t, int64_t,
                                 int, int64_t, int64_t, const int32_t *, const GrpMat *, int);

template <> int lu_small_max_order<z64>() { return 64; }
template <> int lu_small_max_order<c64>() { return 128; }

template <typename T>
void lu_small(hipStream_t s, const GrpMat *grp, int nodes, int count, int64_t pstride,
              int32_t *ipiv, int32_t *info) {
  if (count <= 0) return;
  // persistent: at most four workgroups per compute unit, each looping over matrices
  const unsigned grid = static_cast<unsigned>(std::min(count, 1024));
  hipLaunchKernelGGL((k_lu_small<T, (sizeof(T) == 16 ? 64 : 128)>), dim3(grid), dim3(256), 0, s,
                     grp, nodes, count, pstride, ipiv, info);
}
template void lu_small<z64>(hipStream_t, const GrpMat *, int, int, int64_t, int32_t *, int32_t *);
template void lu_small<c64>(hipStream_t, const GrpMat *, int, int, int64_t, int32_t *, int32_t *);

template <typename T>
void panel_rank(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                int64_t c0, int w1, int w2, const GrpMat *grp, int nodes) {
  const int64_t rows = n - c0 - w1;
  if (w1 <= 0 || w2 <= 0 || w1 > kPU || batch <= 0 || rows <= 0) return;
  hipLaunchKernelGGL((k_panel_rank<T>),
                     dim3(static_cast<unsigned>((rows + 63) / 64), batch, (w2 + kPU - 1) / kPU),
                     dim3(256), 0, s, M, ld, stride, n, c0, w1, w2, grp, nodes);
}
template <typename T>
void panel_solve(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                 int64_t c0, int w1, int w2, const GrpMat *grp, int nodes) {
  if (w1 <= 0 || w2 <= 0 || w1 > 64 || w2 > 64 || batch <= 0) return;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(256), 0, s, M, ld, stride, n, c0, w1, w2, grp, nodes);
  };
  w1 <= kPU ? go(k_panel_solve<T, kPU>) : go(k_panel_solve<T, 64>);
}
template void panel_solve<z64>(hipStream_t, z64 *, int64_t, int64_t, int32_t, int64_t, int64_t, int,
                               int, const GrpMat *, int);
template void panel_solve<c64>(hipStream_t, c64 *, int64_t, int64_t, int32_t, int64_t, int64_t, int,
                               int, const GrpMat *, int);

template <typename T>
void panel_update(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                  int64_t c0, int w1, int w2, const GrpMat *grp, int nodes) {
  if (w1 <= 0 || w2 <= 0 || w1 > kPU || w2 > kPU || batch <= 0) return;
  panel_solve<T>(s, M, ld, stride, batch, n, c0, w1, w2, grp, nodes);
  panel_rank<T>(s, M, ld, stride, batch, n, c0, w1, w2, grp, nodes);
}

// Columns [c0, c0 + w), w <= 64, of each matrix: leaves of eight columns, each
// of which solves its own rows over the rest of a block of `bw` columns and is
// followed by the update of that block's rows below (eight columns deep);
// blocks of 32 are joined by panel_update.  A block of 64 saves that join's two
// launches (about 18 us) and passes over the block's rows 28 times eight columns
// instead of 17: it is taken while a pass over all matrices' rows moves less
// than 8 MB.  Above 8-column leaves' row limit: recursion down to the leaves.
template <typename T>
bool panel_cols(hipStream_t s, T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                int64_t c0, int w, int64_t pk0, int pkb, int32_t *ipiv, int32_t *info,
                const GrpMat *grp, int nodes) {
  const int ib = leaf_max_width<T>(n - c0);
  if (w <= ib) return leaf_lu<T>(s, M, ld, stride, batch, n, c0, w, pk0, pkb, 0, ipiv, info, grp, nodes);
  if (ib < 8) {
    const int w1 = w / 2, w2 = w - w1;
    if (w > 2 * kPU || !panel_cols<T>(s, M, ld, stride, batch, n, c0, w1, pk0, pkb, ipiv, info, grp, nodes))
      return false;
    panel_update<T>(s, M, ld, stride, batch, n, c0, w1, w2, grp, nodes);
    return panel_cols<T>(s, M, ld, stride, batch, n, c0 + w1, w2, pk0, pkb, ipiv, info, grp, nodes);
  }
  const int bw = batch * (n - c0) * static_cast<int64_t>(sizeof(T)) <= (512 << 10) ? 64 : kPU;
  for (int b0 = 0; b0 < w; b0 += bw) {
    const int be = b0 + bw < w ? b0 + bw : w;
    for (int l0 = b0; l0 < be; l0 += 8) {
      const int lw = be - l0 < 8 ? be - l0 : 8, rest = be - l0 - lw;
      if (!leaf_lu<T>(s, M, ld, stride, batch, n, c0 + l0, lw, pk0, pkb, rest, ipiv, info, grp, nodes))
        return false;
      panel_rank<T>(s, M, ld, stride, batch, n, c0 + l0, lw, rest, grp, nodes);
    }
    if (be < w) panel_update<T>(s, M, ld, stride, batch, n, c0 + b0, be - b0, w - be, grp, nodes);
  }
  return true;
}
template bool panel_cols<z64>(hipStream_t, z64 *, int64_t, int64_t, int32_t, int64_t, int64_t, int,
                              int64_t, int, int32_t *, int32_t *, const GrpMat *, int);
template bool panel_cols<c64>(hipStream_t, c64 *, int64_t, int64_t, int32_t, int64_t, int64_t, int,
                              int64_t, int, int32_t *, int32_t *, const GrpMat *, int);

template <typename T>
void diag_block_inverse(hipStream_t s, const T *M, int64_t ld, int64_t stride, int32_t batch,
                        int64_t n, int64_t blk0, int64_t blk1, bool lower, T *out,
                        int64_t out_stride, const GrpMat *grp, int nodes, T *other) {
  if (blk1 <= blk0) return;
  hipLaunchKernelGGL((k_diag_inv<T>), dim3(static_cast<unsigned>(blk1 - blk0), batch, other ? 2 : 1),
                     dim3(256), 0, s, M, ld, stride, n, blk0, lower, out, other, out_stride, grp, nodes);
}
template void diag_block_inverse<z64>(hipStream_t, const z64 *, int64_t, int64_t, int32_t,
                                      int64_t, int64_t, int64_t, bool, z64 *, int64_t,
                                      const GrpMat *, int, z64 *);
template void diag_block_inverse<c64>(hipStream_t, const c64 *, int64_t, int64_t, int32_t,
                                      int64_t, int64_t, int64_t, bool, c64 *, int64_t,
                                      const GrpMat *, int, c64 *);

template <typename T>
void inverse_pairs(hipStream_t s, const T *M, int64_t ld, int64_t stride, int32_t batch, int64_t n,
                   const T *Linv, const T *Uinv, int64_t istride, T *Linv2, T *Uinv2,
                   int64_t istride2) {
  const int64_t nb2 = (n + 127) / 128;
  if (nb2 <= 0 || batch <= 0) return;
  hipLaunchKernelGGL((k_inv_pair<T>), dim3(static_cast<unsigned>(nb2), batch, 2), dim3(256), 0, s, M,
                     ld, stride, n, Linv, Uinv, istride, Linv2, Uinv2, istride2);
}
template void inverse_pairs<z64>(hipStream_t, const z64 *, int64_t, int64_t, int32_t, int64_t,
                                 const z64 *, const z64 *, int64_t, z64 *, z64 *, int64_t);
template void inverse_pairs<c64>(hipStream_t, const c64 *, int64_t, int64_t, int32_t, int64_t,
                                 const c64 *, const c64 *, int64_t, c64 *, c64 *, int64_t);

void perm_from_ipiv(hipStream_t s, const int32_t *ipiv, int32_t *perm, int64_t n, int32_t batch,
                    const GrpMat *grp, int nodes) {
  hipLaunchKernelGGL(k_perm, dim3(batch), dim3(1024), static_cast<unsigned>(n * sizeof(int32_t)), s,
                     ipiv, perm, n, grp, nodes);
}

void fill_i32(hipStream_t s, int32_t *p, int64_t count, int32_t v) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_fill_i32, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s,
                     p, count, v);
}

}  // namespace feast
