// One BM x BN output tile of a complex product on the matrix cores, by 256 threads
// (four wavefronts in a WR x 4 / WR grid).
//
// FP64 and FP32 MFMAs share the vector ALUs' issue: a cycle spent on an address, a bound
// or an operand sum is a cycle without an MFMA (counters: MFMA busy share + 4 cycles
// per vector instruction come to 0.93 to 0.98 of the time).  So:
//   - operands lie in LDS as complex numbers, k-major; a fragment is one 8- or
//     16-byte read, and the sums of the three-product form are made in registers
//     (negations are operand modifiers);
//   - loads and stores are buffer instructions: a uniform base that the scalar unit
//     advances, a byte offset per lane that never changes, and a bound that is an
//     offset past the buffer (reads zero, drops the store);
//   - rows of A and columns of B past the matrix read the last one (their products
//     are not stored), so only a partial last K step has a bound at all.
// And a wavefront must not wait with the matrix cores idle: step kt + 1 goes to the
// other LDS buffer and step kt + 2 is requested at the start of step kt; fragments of
// k group kk + 1 are read before the MFMAs of kk are issued, and those of the next
// step's first group right after the barrier, before the last group's MFMAs
// (sched_barrier keeps the scheduler from undoing either: left alone it waits for
// each LDS read in turn).  64 x 32 tiles: 64 registers a lane in complex64 (eight
// wavefronts a SIMD), 114 in complex128 (four); 64 x 64 is as fast in complex64 and
// 5 % slower in complex128, 128 x 64 8 % slower in both, and 32 columns waste less
// of a ragged N.
//   TFLOP/s (8 flops a complex multiply-add), against tiles of separate planes with
//   a bound on each load: complex64 2048 x 2048 x 256, 32 matrices, 135 -> 170;
//   1024 x 160 x 1024, 32 matrices, 112 -> 163; complex128 2048 x 2048 x 384, 16
//   matrices, 70 -> 86; 1024 x 160 x 1024, 32 matrices, 58 -> 85 (peak of the
//   three-product form 209 and 105).
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"

namespace feast {

enum TileMode {
  kTileGen,  // C = alpha op(A) B + beta C (C read in the epilogue; split-K)
  kTileSub,  // C -= op(A) B: accumulators start from C, MFMAs use -A, plain stores
  kTileShift // C = C0 - (shift[b] A2 - A) B: as kTileSub from C0, A formed in registers
};

// Where a tile's A, B or C lies: 2^31 - 1 bytes from a uniform base (buffer
// instructions, byte offsets), or anywhere (WIDE: pointers, element offsets).
template <typename T, bool WIDE> struct TileSpan;

template <typename T> struct TileSpan<T, false> {
  using off_t = uint32_t;
  static constexpr off_t kOut = 0x80000000u;  // past the buffer: reads zero, drops stores
  __amdgpu_buffer_rsrc_t r;
  __device__ explicit TileSpan(const T *p)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, kOut, 0x00027000)) {}
  __device__ static off_t at(int row, int64_t ld, int col) {
    return (static_cast<uint32_t>(row) * static_cast<uint32_t>(ld) + col) *
           static_cast<uint32_t>(sizeof(T));
  }
  __device__ T load(off_t v, off_t s = 0) const {
    if constexpr (sizeof(T) == 8)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0));
  }
  // (the scalar offset of a 16-byte store goes into the lanes' offset: with a scalar
  // register there the compiler leaves no wait state between the store and a vector
  // write to its data registers, and low words of results were seen overwritten;
  // without one it does.  A lane past the buffer stays past it, s being under 2^31)
  __device__ void store(T x, off_t v, off_t s) const {
    typedef uint32_t words __attribute__((ext_vector_type(sizeof(T) / 4)));
    if constexpr (sizeof(T) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(words, x), r, v, s, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(words, x), r, v + s, 0, 0);
  }
};

template <typename T> struct TileSpan<T, true> {
  using off_t = int64_t;
  static constexpr off_t kOut = -1;
  T *p;
  __device__ explicit TileSpan(const T *q) : p(const_cast<T *>(q)) {}
  __device__ static off_t at(int row, int64_t ld, int col) { return row * ld + col; }
  __device__ T load(off_t v, off_t s = 0) const { return v >= 0 ? p[v + s] : T{}; }
  __device__ void store(T x, off_t v, off_t s) const {
    if (v >= 0) p[v + s] = x;
  }
};

constexpr int kTileM = 64, kTileN = 32;  // the tile of every launch but the two named ones
constexpr int kTileK = 8;
constexpr int kFoldK = 128;  // three-product form: K steps between folds of T1 (power of 2)

// `lin` indexes the tiles x batch x splits of problem d.
//
// M3: three real products per complex one,
//   T1 = (Ar + Ai) Br,  P = -Ai (Br + Bi),  Q = Ar (Bi - Br),
//   Re(AB) = T1 + P,    Im(AB) = T1 + Q
// (its normwise rounding bound is about twice the usual one); otherwise four.
// TA: 0, A is M x K; 2, A is stored K x M and op(A) = A^*.
//
// NG > 1: the workgroup is NG groups of 256 threads, each with LDS of its own, working
// on NG tiles at once.  A group's four wavefronts meet at a barrier of their own (an
// LDS counter, gcount, that each wavefront raises by one per barrier and waits on
// until it reaches *gphase), so the groups do not run in lockstep: while one waits
// for its operands another computes.  A group with no tile of its own passes
// own = false with any valid lin: it stages operands but issues no MFMAs or stores.
template <typename T, int BM, int BN, int WR, int TA, TileMode MODE, bool M3, bool WIDE = false,
          int NG = 1>
__device__ __forceinline__ void gemm_tile(const GemmArgs<T> &d, int64_t lin64, bool own = true,
                                          uint32_t *gcount = nullptr, uint32_t *gphase = nullptr) {
  static_assert(MODE != kTileShift || TA == 0, "shifted operand: C0 - (s A2 - A) B only");
  using Ops = mfma_ops<T>;
  using Span = TileSpan<T, WIDE>;
  using off_t = typename Span::off_t;
  using real = typename Ops::real;
  using acc_t = typename Ops::acc_t;
  constexpr bool SUB = MODE != kTileGen, SHF = MODE == kTileShift;
  constexpr int BK = kTileK, KK = BK / 4;
  constexpr int WC = 4 / WR, WM = BM / WR, WN = BN / WC, FM = WM / 16, FN = WN / 16;
  constexpr int NA = BM * BK / 256, NB = BN * BK / 256;
  static_assert(WM % 16 == 0 && WN % 16 == 0 && BM * BK % 256 == 0 && BN * BK % 256 == 0, "tile");
  static_assert(KK == 2, "fragment buffers");
  // Pitches: the elements that one pass of a store puts down (BK of k by 4 rows in
  // complex64, by 2 in complex128) lie on distinct banks, and so do those of a read
  // (16 consecutive complex numbers of a k row).
  constexpr bool F32 = sizeof(real) == 4;
  constexpr int PA = F32 ? BM + 4 : BM + 2, PB = BN;
  __shared__ T gA[NG][2][BK][PA], gB[NG][2][BK][PB];
  // (NG > 1 runs in a loop over tiles: the thread index passes through an
  // empty asm statement so that the addresses derived from it are formed
  // again in each round instead of being held in registers across the loop)
  int tx = static_cast<int>(threadIdx.x);
  if constexpr (NG > 1) asm volatile("" : "+v"(tx));
  const int gsel = NG > 1 ? __builtin_amdgcn_readfirstlane(tx >> 8) : 0;  // wave-uniform
  auto &sA = gA[gsel];
  auto &sB = gB[gsel];

  const uint32_t tm = static_cast<uint32_t>((d.M + BM - 1) / BM);
  const uint32_t tn = static_cast<uint32_t>((d.N + BN - 1) / BN);
  const uint32_t tiles = tm * tn;
  if (lin64 >= static_cast<int64_t>(tiles) * d.batch * d.splits) return;
  uint32_t lin = static_cast<uint32_t>(lin64);  // (a grid has at most 2^32 - 1 workgroups)
  const uint32_t tile = lin % tiles;
  lin /= tiles;
  const int64_t bidx = lin % d.batch, split = lin / d.batch;
  // tiles in groups of up to 8 tile rows, column by column inside a group:
  // consecutive workgroups share the A row panels of the group (kept in L2)
  // and read each B column panel once per group instead of once per tile row
  constexpr uint32_t G = 8;
  const uint32_t grp = tile / (G * tn), gr0 = grp * G;
  const uint32_t grows = tm - gr0 < G ? tm - gr0 : G, gt = tile - grp * G * tn;
  const int64_t m0 = static_cast<int64_t>(gr0 + gt % grows) * BM;
  const int64_t n0 = static_cast<int64_t>(gt / grows) * BN;
  const int mrem = static_cast<int>(d.M - m0 < BM ? d.M - m0 : BM);
  const int nrem = static_cast<int>(d.N - n0 < BN ? d.N - n0 : BN);
  const int64_t kbeg = split * d.kchunk;
  const int64_t klen = (kbeg + d.kchunk < d.K ? kbeg + d.kchunk : d.K) - kbeg;
  const int nfull = static_cast<int>(klen / BK), tail = static_cast<int>(klen % BK);
  const int nk = nfull + (tail != 0);
  real zr = 0, zi = 0;
  if constexpr (SHF) {
    zr = static_cast<real>(d.shift[bidx].x);
    zi = static_cast<real>(d.shift[bidx].y);
  }

  const int tid = NG > 1 ? (tx & 255) : tx;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WC, wn = wave % WC;
  const int col16 = lane & 15, krow = lane >> 4;
  // barrier of the threads that share this tile's LDS
  auto tile_sync = [&]() {
    if constexpr (NG == 1) {
      __syncthreads();
    } else {
      *gphase += 4;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) __hip_atomic_fetch_add(gcount, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      while (__hip_atomic_load(gcount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < *gphase)
        __builtin_amdgcn_s_sleep(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
  };
  // a wavefront whose whole output block lies outside C (ragged last tile)
  // stages operands and meets the barriers but issues no MFMAs
  const bool live = own && wm * WM < mrem && wn * WN < nrem;

  // This thread's elements of a K step.  A: TA = 0, BK lanes read one row's BK
  // consecutive elements; TA = 2, consecutive lanes the consecutive rows of op(A).
  // B: consecutive lanes consecutive columns.
  auto ak = [&](int i) { return TA == 0 ? tid % BK : (tid + 256 * i) / BM; };
  auto ar = [&](int i) { return TA == 0 ? tid / BK + (256 / BK) * i : (tid + 256 * i) % BM; };
  auto bk = [&](int i) { return (tid + 256 * i) / BN; };
  auto bc = [&](int i) { return (tid + 256 * i) % BN; };
  const T *ua = d.A + bidx * d.sA + (TA == 0 ? m0 * d.lda + kbeg : kbeg * d.lda + m0);
  const T *ua2 = SHF ? d.A2 + bidx * d.sA + m0 * d.lda + kbeg : nullptr;
  const T *ub = d.B + bidx * d.sB + kbeg * d.ldb + n0;
  const int64_t stepa = TA == 0 ? BK : BK * d.lda, stepb = BK * d.ldb;
  off_t oa[NA], ob[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int r = ar(i) < mrem ? ar(i) : mrem - 1;
    oa[i] = TA == 0 ? Span::at(r, d.lda, ak(i)) : Span::at(ak(i), d.lda, r);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) ob[i] = Span::at(bk(i), d.ldb, bc(i) < nrem ? bc(i) : nrem - 1);
  T ra[NA], rb[NB], ra2[SHF ? NA : 1];
  int kl = 0;  // the next K step to load
  auto gload = [&]() {
    const Span qa(ua), qa2(ua2), qb(ub);
    if (kl < nfull) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        ra[i] = qa.load(oa[i]);
        if constexpr (SHF) ra2[i] = qa2.load(oa[i]);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) rb[i] = qb.load(ob[i]);
    } else {  // the last, partial step: zeros past K
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const off_t o = ak(i) < tail ? oa[i] : Span::kOut;
        ra[i] = qa.load(o);
        if constexpr (SHF) ra2[i] = qa2.load(o);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) rb[i] = qb.load(bk(i) < tail ? ob[i] : Span::kOut);
    }
    ++kl;
    ua += stepa;
    if constexpr (SHF) ua2 += stepa;
    ub += stepb;
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      T v = ra[i];
      if constexpr (SHF) {
        v.x = zr * ra2[i].x - zi * ra2[i].y - ra[i].x;
        v.y = zr * ra2[i].y + zi * ra2[i].x - ra[i].y;
      }
      if constexpr (TA == 2) v.y = -v.y;
      sA[buf][ak(i)][ar(i)] = v;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) sB[buf][bk(i)][bc(i)] = rb[i];
  };
  if (nk > 0) gload();

  // element (a, b, r) of this lane's part of C, outside C past the span
  constexpr int RS = F32 ? 1 : 4;  // out_row(lane, r + 1) - out_row(lane, r)
  const int crow = wm * WM + Ops::out_row(lane, 0), ccol = wn * WN + col16;
  auto cin = [&](int a, int b, int r, off_t o) {
    return crow + a * 16 + r * RS < mrem && ccol + b * 16 < nrem ? o : Span::kOut;
  };
  acc_t cr[FM][FN], ci[FM][FN], t1[M3 ? FM : 1][M3 ? FN : 1];
  {
    const int64_t ld = SHF ? d.ldc0 : d.ldc;
    const Span q(SHF ? d.C0 + bidx * d.sC0 + m0 * ld + n0 : d.C + bidx * d.sC + m0 * ld + n0);
    const off_t o = Span::at(crow, ld, ccol);
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int b = 0; b < FN; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          T v{};
          if constexpr (SUB) v = q.load(cin(a, b, r, o), Span::at(a * 16 + r * RS, ld, b * 16));
          cr[a][b][r] = v.x;
          ci[a][b][r] = v.y;
          if constexpr (M3) t1[a][b][r] = 0;
        }
  }

  T fa[2][FM], fb[2][FN];
  auto frags = [&](int buf, int kk, int o) {
#pragma unroll
    for (int a = 0; a < FM; ++a) fa[o][a] = sA[buf][kk * 4 + krow][wm * WM + a * 16 + col16];
#pragma unroll
    for (int b = 0; b < FN; ++b) fb[o][b] = sB[buf][kk * 4 + krow][wn * WN + b * 16 + col16];
  };
  // (sweeps over all tiles: an accumulator is reused only after every other
  // accumulator of the wavefront has been issued once)
  auto mul = [&](int o) {
    if constexpr (M3) {
      real as[FM], bs[FN], bd[FN];
#pragma unroll
      for (int a = 0; a < FM; ++a) as[a] = SUB ? -fa[o][a].x - fa[o][a].y : fa[o][a].x + fa[o][a].y;
#pragma unroll
      for (int b = 0; b < FN; ++b) {
        bs[b] = SUB ? fb[o][b].x + fb[o][b].y : -fb[o][b].x - fb[o][b].y;
        bd[b] = SUB ? fb[o][b].x - fb[o][b].y : fb[o][b].y - fb[o][b].x;
      }
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) t1[a][b] = Ops::mma(as[a], fb[o][b].x, t1[a][b]);
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) cr[a][b] = Ops::mma(fa[o][a].y, bs[b], cr[a][b]);
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) ci[a][b] = Ops::mma(fa[o][a].x, bd[b], ci[a][b]);
    } else {
      // SUB accumulates (-A) B:  Cr += (-Ar) Br - (-Ai) Bi, Ci += (-Ar) Bi + (-Ai) Br
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          const real x = SUB ? -fa[o][a].x : fa[o][a].x;
          cr[a][b] = Ops::mma(x, fb[o][b].x, cr[a][b]);
          ci[a][b] = Ops::mma(x, fb[o][b].y, ci[a][b]);
        }
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) {
          const real y = SUB ? -fa[o][a].y : fa[o][a].y;
          cr[a][b] = Ops::mma(-y, fb[o][b].y, cr[a][b]);
          ci[a][b] = Ops::mma(y, fb[o][b].x, ci[a][b]);
        }
    }
  };
  // T1 folded into both parts every kFoldK steps of K: the shared term
  // then never sums more than kFoldK products before it meets P and Q,
  // whatever the launch's K (long K ranges otherwise let T1 and P grow
  // far beyond their difference, and the complex64 factors lose digits)
  auto fold = [&]() {
    if constexpr (M3) {
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            cr[a][b][r] += t1[a][b][r];
            ci[a][b][r] += t1[a][b][r];
            t1[a][b][r] = 0;
          }
    }
  };
  // K step kt, in LDS buffer `buf` with its first fragments read
  auto step = [&](int kt, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    if (kt + 1 < nk) sstore(buf ^ 1);  // (last read before the barrier of step kt - 1)
    if (kt + 2 < nk) gload();
    if (live) {
      frags(buf, 1, 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    tile_sync();
    if (live) {
      if (kt + 1 < nk) frags(buf ^ 1, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      mul(1);
      __builtin_amdgcn_sched_barrier(0);
      // (the last fold is the epilogue's)
      if (M3 && ((kt + 1) & (kFoldK / BK - 1)) == 0 && kt + 1 < nk) fold();
    }
  };
  if (nk > 0) {
    sstore(0);
    if (nk > 1) gload();
    tile_sync();
    if (live) frags(0, 0, 0);
    for (int kt = 0; kt < nk; kt += 2) {  // two steps a turn: the buffer index is a constant
      step(kt, std::integral_constant<int, 0>{});
      if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{});
    }
  }
  if (!live) return;
  fold();

  // split-K partials go to the workspace (M x N, contiguous)
  const bool part = !SUB && d.splits > 1;
  const int64_t ld = part ? d.N : d.ldc;
  const Span q((part ? d.work + (split * d.batch + bidx) * d.M * d.N : d.C + bidx * d.sC) + m0 * ld + n0);
  const off_t o = Span::at(crow, ld, ccol);
  const real alr = static_cast<real>(d.alpha.x), ali = static_cast<real>(d.alpha.y);
  const real ber = static_cast<real>(d.beta.x), bei = static_cast<real>(d.beta.y);
  const bool use_beta = !part && (ber != 0 || bei != 0);
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const off_t v = cin(a, b, r, o), s = Span::at(a * 16 + r * RS, ld, b * 16);
        T x;
        x.x = cr[a][b][r];
        x.y = ci[a][b][r];
        if constexpr (!SUB) {
          const real xr = x.x, xi = x.y;
          x.x = alr * xr - ali * xi;
          x.y = alr * xi + ali * xr;
          if (use_beta) {
            const T c = q.load(v, s);
            x.x += ber * c.x - bei * c.y;
            x.y += ber * c.y + bei * c.x;
          }
        }
        q.store(x, v, s);
      }
}

// Whether every offset within a tile of the launch fits a 2^31 - 1 byte span.
template <typename T> bool tile_spans_fit(const GemmArgs<T> &d, int ta, int bm) {
  const int64_t lim = (int64_t{1} << 31) / static_cast<int64_t>(sizeof(T));
  return (ta == 0 ? bm * d.lda + kTileK : kTileK * d.lda + bm) < lim &&
         kTileK * d.ldb + 64 < lim && bm * std::max(d.ldc, d.N) + 64 < lim &&
         (!d.C0 || bm * d.ldc0 + 64 < lim);
}

}  // namespace feast
