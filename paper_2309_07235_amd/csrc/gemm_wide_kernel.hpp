// LDS-tiled MFMA GEMM for the products whose schedule the library picks itself: the products of 3mm (paper,
// 3mm_basic listing) and those of the solves with many right-hand sides.  A schedule that the caller names runs on
// gemm_kernel.
//
// What bounds gemm_kernel on these shapes is the round trip of a k-slab: its loads are issued one slab ahead, and with
// the two to four workgroups per compute unit that such products have, a slab is multiplied (0.2 - 0.9 us) before the
// next one has arrived.  Its fragment reads are also 8 bytes each (4 in fp32), its LDS writes too.  Here
//   - two slabs are in flight: slab s + 2 is requested before slab s is multiplied, into the register set that slab s
//     left, and slab s + 1 goes from the other set to LDS half way through the multiplication;
//   - a slab is 128 bytes of k, and k is dealt to the lanes so that the left operand's values of a lane are one run:
//     lane group l4 (the k index of an MFMA) takes k = KPL l4 + kk in step kk of KPL, two 16-byte LDS reads a slab and
//     row block.  The row stride is odd in units of 16 bytes, so the 8 rows one access cycle serves use all banks (left
//     as conflicts are 17 - 22 % of the LDS cycles, by counter, with the matrix pipes busy 81 - 83 % of the time);
//   - where a wave has two column blocks (the 64 x 64 and 128 x 64 tiles) they are interleaved, block b taking the columns
//     2 l15 + b, so the right operand is read and C is read and stored two elements at a time;
//   - a ragged tile runs the same pipeline: a row past the edge is clamped to the last one, the run of columns across it
//     reads on (both only reach results that are not stored); only the last slab is masked, on the way from the registers
//     to LDS.  A mask where a value is loaded makes it wait for the load: with that, a width that is not a multiple of 16
//     bytes took up to 1.67 times as long as on gemm_kernel (Cholesky solve N = 8192, 255 right-hand sides, fp32: 2095 us,
//     now 1015; LU solve N = 4001, 301, fp64: 1180 us, now 675).  Moving the run across the edge to its place in every
//     slab keeps both forms of the loop in registers: 108 instead of 72 in a 64 x 64 tile, a workgroup less per unit.
// The two larger tiles have eight waves, two on each SIMD, which cover each other's barrier, the smaller ones four, and
// more workgroups to a unit.  Measured, back to back, gemm_kernel with its default schedule against this:
// 4096 x 4096 x 1024 57 against 71 TFLOP/s in fp64 (of 78.6), 106 against 131 in fp32; 3mm extralarge fp64 848 against
// 713 us, large fp32 130 against 64.5, with every dimension one more 130 against 65.  On its first form, deeper slabs
// (256 bytes) were 5 % slower, shallower ones (64 bytes) 2 - 10 %, 16 waves per 64 x 64 tile 10 %.
#pragma once
#include <type_traits>
#include "gemm_kernel.hpp"

namespace dla {

// runs of N elements as one access that needs no more alignment than one element
template <typename T, int N>
struct WideRun;
template <typename T>
struct WideRun<T, 1> {
  typedef T type __attribute__((ext_vector_type(1)));
};
template <>
struct WideRun<double, 2> {
  typedef double type __attribute__((ext_vector_type(2), aligned(8)));
};
template <>
struct WideRun<float, 2> {
  typedef float type __attribute__((ext_vector_type(2), aligned(4)));
};
template <>
struct WideRun<float, 4> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <typename T>
struct WideVec {  // 16 bytes
  static constexpr int PER = 16 / (int)sizeof(T);
  using v16 = typename WideRun<T, PER>::type;
};

// F: adjacent blocks one lane serves from one run of contiguous elements
constexpr int wide_run(int f) { return f % 2 == 0 ? 2 : 1; }

template <typename T, int WM, int WN, int FM, int FN, int TK, bool AT>
struct WideShape {
  static constexpr int TM = WM * FM * 16, TN = WN * FN * 16;
  static constexpr int NT = WM * WN * 64;
  static constexpr int PER = WideVec<T>::PER;
  static constexpr int SA = AT ? TM : TK + PER;      // LDS row stride of the left operand
  static constexpr int SB = TN;
  static constexpr int A_ELEMS = AT ? TK * SA : TM * SA;
  static constexpr int B_ELEMS = TK * SB;
  static constexpr int STAGE = A_ELEMS + B_ELEMS;
  static constexpr int BYTES = 2 * STAGE * (int)sizeof(T);
};

// x, as a value that the compiler cannot compute ahead: what only the last slab needs is worked out there, instead of
// being kept in registers beside the loop.
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A ROWS x COLS tile (COLS contiguous in memory) in passes of NT threads, 16 bytes per thread and pass.
template <typename T, int ROWS, int COLS, int NT>
struct WideLoader {
  static constexpr int PER = WideVec<T>::PER;
  static constexpr int VPR = COLS / PER;
  static constexpr int TOTAL = ROWS * VPR;
  static constexpr int ITER = TOTAL / NT;
  static_assert(COLS % PER == 0, "tile width");
  static __device__ __forceinline__ int row_of(int idx) { return idx / VPR; }
  static __device__ __forceinline__ int col_of(int idx) { return (idx % VPR) * PER; }
};

// The run that began `by` elements (less than a run) before its place: element e to the front of it is element e + by.
// What it holds past the edge is not used.
template <typename T>
__device__ __forceinline__ typename WideVec<T>::v16 wide_move(typename WideVec<T>::v16 x, int by) {
  if constexpr (WideVec<T>::PER == 2) {
    x[0] = by != 0 ? x[1] : x[0];
  } else {
    const bool one = (by & 1) != 0, two = (by & 2) != 0;
    x[0] = one ? x[1] : x[0];
    x[1] = one ? x[2] : x[1];
    x[2] = one ? x[3] : x[2];
    x[0] = two ? x[2] : x[0];
    x[1] = two ? x[3] : x[1];
  }
  return x;
}

// Tile (ti, tj) of product P, by the whole workgroup.  OP_NEGATE: C = -A*B.  Off: the type of element offsets inside a tile.
constexpr int OP_NEGATE = 100;
template <typename T, int WM, int WN, int FM, int FN, int TK, int OP, typename Off = uint32_t>
__device__ __forceinline__ void gemm_wide_tile(const GemmProblem<T>& P, const int ti, const int tj, T* const smem) {
  constexpr bool AT = OP == OP_SUB_TN, SUB = OP != OP_ASSIGN, ONTO = SUB && OP != OP_NEGATE;
  using S = WideShape<T, WM, WN, FM, FN, TK, AT>;
  constexpr int TM = S::TM, TN = S::TN, NT = S::NT, PER = S::PER;
  constexpr int KPL = TK / 4;  // k-steps of a slab = k values per lane
  constexpr int RA = AT ? wide_run(FM) : 1, RB = wide_run(FN);
  using acc_t = typename Mfma<T>::acc_t;
  using V = typename WideVec<T>::v16;
  using R = typename WideRun<T, RB>::type;  // what a lane holds of a row of C, in one access
  using LA = WideLoader<T, AT ? TK : TM, AT ? TM : TK, NT>;
  using LB = WideLoader<T, TK, TN, NT>;
  const int m0 = ti * TM, n0 = tj * TN;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, l4 = lane >> 4;
  const int wm0 = (wave / WN) * (FM * 16), wn0 = (wave % WN) * (FN * 16);
  const int M = P.M, N = P.N, K = P.K;
  const int64_t lda = P.lda, ldb = P.ldb, ldc = P.ldc;
  const bool full_mn = m0 + TM <= M && n0 + TN <= N;

  // row of the tile held by index i of row block a, column held by lane l15 of column block b
  auto row_at = [&](int a, int i) { return wm0 + (a / RA) * 16 * RA + i * RA + a % RA; };
  const int coll = wn0 + l15 * RB;
  auto col_at = [&](int b) { return coll + (b / RB) * 16 * RB + b % RB; };

  acc_t acc[FM][FN];
  T* const Ct = P.C + (int64_t)m0 * ldc + n0;
  if constexpr (ONTO) {
    if (full_mn) {
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int b = 0; b < FN; b += RB) {
            const R w = *reinterpret_cast<const R*>(Ct + (int64_t)row_at(a, Mfma<T>::row_of(v, lane)) * ldc + col_at(b));
#pragma unroll
            for (int e = 0; e < RB; ++e) acc[a][b + e][v] = w[e];
          }
    } else {
      const int rmax = M - 1 - m0, cmax = N - 1 - n0;
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = row_at(a, Mfma<T>::row_of(v, lane));
          const T* const p = Ct + (int64_t)(r < rmax ? r : rmax) * ldc;
#pragma unroll
          for (int b = 0; b < FN; ++b) acc[a][b][v] = p[col_at(b) < cmax ? col_at(b) : cmax];
        }
    }
  } else {
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int b = 0; b < FN; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
  }

  // ---- operand loads: 16-byte runs.  Rows past the edge are clamped, runs past it to the one that straddles it.  That
  // one reads on into what follows its row in memory; only in the last row might there be nothing, so a tile with a
  // straddling run loads its last slab as a partial one.
  const T* const Ag = AT ? P.A : P.A + (int64_t)m0 * lda;
  const T* const Bg = P.B;
  static_assert(LA::TOTAL % NT == 0 && LB::TOTAL % NT == 0 && NT % LA::VPR == 0 && NT % LB::VPR == 0, "whole passes, one column per thread");
  const bool narrow_a = AT && M < PER, narrow_b = N < PER;  // rows shorter than a run
  const bool straddle = (AT && m0 + TM > M && M % PER != 0) || (n0 + TN > N && N % PER != 0);
  Off aoff[LA::ITER], boff[LB::ITER];                  // element offsets of slab 0
#pragma unroll
  for (int it = 0; it < LA::ITER; ++it) {
    const int r = LA::row_of(tid + it * NT), c = LA::col_of(tid), last = (M - 1) / PER * PER;
    if constexpr (AT) aoff[it] = (Off)r * (Off)lda + (Off)(m0 + c < last ? m0 + c : last);
    else aoff[it] = (Off)(m0 + r < M ? r : M - 1 - m0) * (Off)lda + (Off)c;
  }
#pragma unroll
  for (int it = 0; it < LB::ITER; ++it) {
    const int r = LB::row_of(tid + it * NT), c = n0 + LB::col_of(tid), last = (N - 1) / PER * PER;
    boff[it] = (Off)r * (Off)ldb + (Off)(c < last ? c : last);
  }
  V ra[2][LA::ITER], rb[2][LB::ITER];
  auto load_full = [&](auto sc, int s) __attribute__((always_inline)) {
    constexpr int X = decltype(sc)::value;
    const T* const pa = AT ? Ag + (int64_t)s * TK * lda : Ag + (int64_t)s * TK;
    const T* const pb = Bg + (int64_t)s * TK * ldb;
#pragma unroll
    for (int it = 0; it < LA::ITER; ++it) ra[X][it] = *reinterpret_cast<const V*>(pa + aoff[it]);
#pragma unroll
    for (int it = 0; it < LB::ITER; ++it) rb[X][it] = *reinterpret_cast<const V*>(pb + boff[it]);
  };
  // A partial slab, a tile's last one with a straddling run, all slabs of a narrow operand: k past the end is clamped, a
  // run past the end of its row starts at the row's last whole run (an operand narrower than a run: element by element,
  // clamped to its last column).  What that brings too much or in the wrong place is seen to in stash: a mask here would
  // make each load wait for the one before it.
  auto load_tail = [&](auto sc, int s) __attribute__((always_inline)) {
    constexpr int X = decltype(sc)::value;
    const int kv = K - s * TK, t = here(tid);
    const T* const pa = AT ? Ag + (int64_t)s * TK * lda : Ag + (int64_t)s * TK;
    const T* const pb = Bg + (int64_t)s * TK * ldb;
#pragma unroll
    for (int it = 0; it < LA::ITER; ++it) {
      const int r = LA::row_of(t + it * NT), c = LA::col_of(t);
      if constexpr (AT) {
        const T* const q = pa + (Off)(r < kv ? r : kv - 1) * (Off)lda;
        if (!narrow_a) {
          ra[X][it] = *reinterpret_cast<const V*>(q + (m0 + c < M - PER ? m0 + c : M - PER));
        } else {
#pragma unroll
          for (int e = 0; e < PER; ++e) ra[X][it][e] = q[c + e < M ? c + e : M - 1];
        }
      } else {
        const T* const q = pa + (Off)(m0 + r < M ? r : M - 1 - m0) * (Off)lda;
#pragma unroll
        for (int e = 0; e < PER; ++e) ra[X][it][e] = q[c + e < kv ? c + e : kv - 1];
      }
    }
#pragma unroll
    for (int it = 0; it < LB::ITER; ++it) {
      const int r = LB::row_of(t + it * NT), c = n0 + LB::col_of(t);
      const T* const q = pb + (Off)(r < kv ? r : kv - 1) * (Off)ldb;
      if (!narrow_b) {
        rb[X][it] = *reinterpret_cast<const V*>(q + (c < N - PER ? c : N - PER));
      } else {
#pragma unroll
        for (int e = 0; e < PER; ++e) rb[X][it][e] = q[c + e < N ? c + e : N - 1];
      }
    }
  };
  // registers to LDS.  TAIL: loaded by load_tail; the straddling run moves to its place, and k past the end becomes zero in
  // both operands, since what a clamped address brought may be anything.
  auto stash = [&](auto sc, auto tail, int buf, int s) __attribute__((always_inline)) {
    constexpr int X = decltype(sc)::value;
    constexpr bool TAIL = decltype(tail)::value;
    T* const sa = smem + buf * S::STAGE;
    T* const sb = sa + S::A_ELEMS;
    const int kv = K - s * TK, t = TAIL ? here(tid) : tid;
#pragma unroll
    for (int it = 0; it < LA::ITER; ++it) {
      V x = ra[X][it];
      const int r = LA::row_of(t + it * NT), c = LA::col_of(t);
      if constexpr (TAIL) {
        if (AT && !narrow_a) x = wide_move<T>(x, m0 + c < M - PER ? 0 : m0 + c - (M - PER));
#pragma unroll
        for (int e = 0; e < PER; ++e) x[e] = (AT ? r : c + e) < kv ? x[e] : T(0);
      }
      *reinterpret_cast<__attribute__((aligned(16))) V*>(sa + r * S::SA + c) = SUB ? -x : x;
    }
#pragma unroll
    for (int it = 0; it < LB::ITER; ++it) {
      V x = rb[X][it];
      const int r = LB::row_of(t + it * NT), c = LB::col_of(t);
      if constexpr (TAIL) {
        if (!narrow_b) x = wide_move<T>(x, n0 + c < N - PER ? 0 : n0 + c - (N - PER));
#pragma unroll
        for (int e = 0; e < PER; ++e) x[e] = r < kv ? x[e] : T(0);
      }
      *reinterpret_cast<__attribute__((aligned(16))) V*>(sb + r * S::SB + c) = x;
    }
  };
  // k of step kk is KPL * l4 + kk in both operands: a lane's left-operand values of a slab are contiguous
  auto multiply = [&](int buf, auto half) __attribute__((always_inline)) {
    constexpr int H = decltype(half)::value;
    const T* const sa = smem + buf * S::STAGE;
    const T* const sb = sa + S::A_ELEMS;
    const T* const pa = AT ? sa + (KPL * l4) * S::SA + wm0 + l15 * RA : sa + (wm0 + l15) * S::SA + KPL * l4;
    const T* const pb = sb + (KPL * l4) * S::SB + coll;
#pragma unroll
    for (int kk = H * (KPL / 2); kk < (H + 1) * (KPL / 2); ++kk) {
      T fa[FM], fb[FN];
#pragma unroll
      for (int a = 0; a < FM; ++a) fa[a] = AT ? pa[kk * S::SA + (a / RA) * 16 * RA + a % RA] : pa[a * 16 * S::SA + kk];
#pragma unroll
      for (int b = 0; b < FN; ++b) fb[b] = pb[kk * S::SB + (b / RB) * 16 * RB + b % RB];
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = Mfma<T>::mma(fa[a], fb[b], acc[a][b]);
    }
  };
  using c0 = std::integral_constant<int, 0>;
  using c1 = std::integral_constant<int, 1>;
  const int nslab = (K + TK - 1) / TK;
  const int nrun = narrow_a || narrow_b ? 0 : (straddle ? K - 1 : K) / TK;  // slabs that load_full loads
  auto load_any = [&](auto sc, int s) __attribute__((always_inline)) {
    if (s < nrun) load_full(sc, s);
    else if (s < nslab) load_tail(sc, s);
  };
  auto stash_any = [&](auto sc, int buf, int s) __attribute__((always_inline)) {
    if (s < nrun) stash(sc, std::false_type{}, buf, s);
    else if (s < nslab) stash(sc, std::true_type{}, buf, s);
  };
  load_any(c0{}, 0);
  load_any(c1{}, 1);
  stash_any(c0{}, 0, 0);
  lds_barrier();
  int s = 0;
  // fp32: the loads stay in front of the multiplication.  The compiler otherwise moves them behind it, which leaves one slab
  // in flight (4 % slower; C = A*B in the larger tiles is as fast).  In fp64 they stay there by themselves.
  auto in_order = [] { if constexpr (sizeof(T) == 4 && (SUB || FN == 1)) __builtin_amdgcn_sched_barrier(0); };
  for (; s + 3 < nrun; s += 2) {
    load_full(c0{}, s + 2);
    in_order();
    multiply(0, c0{});
    stash(c1{}, std::false_type{}, 1, s + 1);
    multiply(0, c1{});
    lds_barrier();
    load_full(c1{}, s + 3);
    in_order();
    multiply(1, c0{});
    stash(c0{}, std::false_type{}, 0, s + 2);
    multiply(1, c1{});
    lds_barrier();
  }
  for (; s < nslab; s += 2) {
    load_any(c0{}, s + 2);
    multiply(0, c0{});
    stash_any(c1{}, 1, s + 1);
    multiply(0, c1{});
    lds_barrier();
    if (s + 1 >= nslab) break;
    load_any(c1{}, s + 3);
    multiply(1, c0{});
    stash_any(c0{}, 0, s + 2);
    multiply(1, c1{});
    lds_barrier();
  }

  auto store_to = [&](T* const D, int64_t ldd) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = row_at(a, Mfma<T>::row_of(v, lane));
#pragma unroll
        for (int b = 0; b < FN; b += RB) {
          const int c = col_at(b);
          T* const p = D + (int64_t)r * ldd + c;
          if (full_mn) {
            R w;
#pragma unroll
            for (int e = 0; e < RB; ++e) w[e] = acc[a][b + e][v];
            *reinterpret_cast<R*>(p) = w;
          } else {
#pragma unroll
            for (int e = 0; e < RB; ++e)
              if (m0 + r < M && n0 + c + e < N) p[e] = acc[a][b + e][v];
          }
        }
      }
  };
  store_to(Ct, ldc);
  if (P.C2) store_to(P.C2 + (int64_t)m0 * P.ldc2 + n0, P.ldc2);
}

template <typename T, int WM, int WN, int FM, int FN, int TK, int OP>
__global__ void __launch_bounds__(WM * WN * 64) gemm_wide_kernel(const GemmGroup<T> g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_contiguous_id((int)blockIdx.x, g.total_tiles);
  int pi = 0;
#pragma unroll
  for (int q = 1; q < kMaxGroup; ++q)
    if (q < g.nprob && logical >= g.prob[q].tile_begin) pi = q;
  const GemmProblem<T>& P = g.prob[pi];
  const int local = logical - P.tile_begin;
  gemm_wide_tile<T, WM, WN, FM, FN, TK, OP>(P, local / P.tiles_n, local % P.tiles_n, reinterpret_cast<T*>(smem_raw));
}

}  // namespace dla
