// Panel-phase kernels of the blocked right-looking factorisations (paper,
// Section "Linear Algebra Benchmarks": A = L*U without pivoting, A = L*L^T):
//
//   diag_kernel   one workgroup factors the b x b diagonal block (b <= 128) held
//                 in LDS, in stages of 16 columns: a wavefront-level 16 x 16
//                 factorisation in registers (one matrix row per lane, pivot row
//                 broadcast with DPP row_newbcast), the 16-wide inner panels by
//                 substitution, one column or row per lane, MFMA for the inner
//                 trailing update.  The identity rides along as 16 more columns of
//                 the panel and comes out as the sub-block's inverse, which goes to
//                 the workspace.
// What bounds it is the chain factor -> panels -> next sub-block's update -> factor of its eight stages.  fp64
// multiply-adds are not the cost (4 cycles each, dependent or not); wait states, selects and compares around them and LDS
// traffic are.  Measured on whole calls, against DPP multiply-adds with wait states of their own, pivots tested in every
// step, inverses and the store behind the last stage, and the first sub-block factored only once the whole block has
// arrived: N = 128 LU fp64 42.0 -> 37.2 us, Cholesky fp64 44.7 -> 38.9, fp32 40.3 -> 33.6; LU N = 4000 1888 -> 1820.
// Panels as products with explicit inverses of 4 x 4 blocks on MFMA are no faster (39.8, 39.8, 34.0, 1853) and not
// substitution: their backward error grows with the condition of these blocks (LU of a kernel matrix of order 33 and
// condition 1e10: 372 eps against 1), and 0 * NaN carries a breakdown into columns in front of it.
// The panel solves and the look-ahead head update, which consume those inverses,
// live in head_kernel.hpp.
#pragma once
#include <type_traits>
#include "dla_common.hpp"

namespace dla {

constexpr int kNbMax = 128;            // largest block size
constexpr int kIb = 16;                // inner block = one MFMA block
constexpr int kSld = kNbMax + 1;       // odd LDS row stride of the diagonal block
constexpr int kDiagThreads = 512;
constexpr int kBlk = kIb * (kIb + 1);  // 16 x 17: one padded 16 x 16 sub-block in LDS

enum FactorKind { KIND_LU = 0, KIND_CHOL = 1 };

template <int I, int N, typename F>
__device__ inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Value of lane K of the caller's 16-lane row, for every lane of that row (DPP row_newbcast).
template <int K>
__device__ inline double row_bcast(double x) {
  return __builtin_amdgcn_update_dpp(x, x, 0x150 + K, 0xF, 0xF, true);  // every lane is written: no 'old' value needed
}
template <int K>
__device__ inline float row_bcast(float x) {
  return __builtin_amdgcn_update_dpp(x, x, 0x150 + K, 0xF, 0xF, true);
}

// acc -= (value of src in lane K of the caller's 16-lane row) * m, as DPP multiply-adds: the
// negation is a source modifier of the instruction, so it adds nothing to a dependent chain.
// The two wait states a DPP read needs after a VALU write of its source are part of the statement.
// They cost a wavefront more than the multiply-add itself (16 cycles for the pair, 6.3 per multiply-add when
// four share one s_nop), so the runs below issue up to four in a statement, where no source is written by an
// earlier instruction of it.  lu16: 2520 -> 2092 cycles, with the pivot tests taken out as well.
#define DLA_FNMAC_BCAST(T, OP)                                                                                \
  template <int K>                                                                                            \
  __device__ inline void fnmac_bcast(T& acc, T src, T m) {                                                    \
    asm("s_nop 1\n\t" OP " %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"                            \
        : "+v"(acc)                                                                                           \
        : "v"(src), "v"(m), "n"(K));                                                                          \
  }                                                                                                           \
  /* accumulators that are their own source: a_q -= a_q[lane K] * m */                                        \
  template <int K>                                                                                            \
  __device__ inline void fnmac_self2(T& a0, T& a1, T m) {                                                     \
    asm("s_nop 1\n\t" OP " %0, -%0, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1)                                                                                \
        : "v"(m), "n"(K));                                                                                    \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_self3(T& a0, T& a1, T& a2, T m) {                                              \
    asm("s_nop 1\n\t" OP " %0, -%0, %3 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%1, %3 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%2, %3 row_newbcast:%4 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2)                                                                     \
        : "v"(m), "n"(K));                                                                                    \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_self4(T& a0, T& a1, T& a2, T& a3, T m) {                                       \
    asm("s_nop 1\n\t" OP " %0, -%0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %3, -%3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)                                                          \
        : "v"(m), "n"(K));                                                                                    \
  }                                                                                                           \
  /* accumulators and one source, adjacent lanes: a_q -= src[lane K + q] * m */                               \
  template <int K>                                                                                            \
  __device__ inline void fnmac_lanes2(T& a0, T& a1, T src, T m) {                                             \
    asm("s_nop 1\n\t" OP " %0, -%2, %3 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1)                                                                                \
        : "v"(src), "v"(m), "n"(K), "n"(K + 1));                                                              \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_lanes3(T& a0, T& a1, T& a2, T src, T m) {                                      \
    asm("s_nop 1\n\t" OP " %0, -%3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%3, %4 row_newbcast:%7 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2)                                                                     \
        : "v"(src), "v"(m), "n"(K), "n"(K + 1), "n"(K + 2));                                                  \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_lanes4(T& a0, T& a1, T& a2, T& a3, T src, T m) {                               \
    asm("s_nop 1\n\t" OP " %0, -%4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %3, -%4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)                                                          \
        : "v"(src), "v"(m), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3));                                      \
  }                                                                                                           \
  /* accumulators and sources, one lane: a_q -= s_q[lane K] * m */                                            \
  template <int K>                                                                                            \
  __device__ inline void fnmac_each2(T& a0, T& a1, T s0, T s1, T m) {                                         \
    asm("s_nop 1\n\t" OP " %0, -%2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1)                                                                                \
        : "v"(s0), "v"(s1), "v"(m), "n"(K));                                                                  \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_each3(T& a0, T& a1, T& a2, T s0, T s1, T s2, T m) {                            \
    asm("s_nop 1\n\t" OP " %0, -%3, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%4, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%5, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2)                                                                     \
        : "v"(s0), "v"(s1), "v"(s2), "v"(m), "n"(K));                                                         \
  }                                                                                                           \
  template <int K>                                                                                            \
  __device__ inline void fnmac_each4(T& a0, T& a1, T& a2, T& a3, T s0, T s1, T s2, T s3, T m) {               \
    asm("s_nop 1\n\t" OP " %0, -%4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"                        \
        OP " %1, -%5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %2, -%6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"                                      \
        OP " %3, -%7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"                                          \
        : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)                                                          \
        : "v"(s0), "v"(s1), "v"(s2), "v"(s3), "v"(m), "n"(K));                                                \
  }
DLA_FNMAC_BCAST(double, "v_fmac_f64_dpp")
DLA_FNMAC_BCAST(float, "v_fmac_f32_dpp")
#undef DLA_FNMAC_BCAST

// Runs over the columns J0 .. J1-1 of a 16-element row:
// a[j] -= a[j][lane K] * m
template <int K, int J0, int J1, typename T>
__device__ inline void fnmac_run_self(T (&a)[16], T m) {
  constexpr int N = J1 - J0;
  if constexpr (N >= 4) {
    fnmac_self4<K>(a[J0], a[J0 + 1], a[J0 + 2], a[J0 + 3], m);
    fnmac_run_self<K, J0 + 4, J1>(a, m);
  } else if constexpr (N == 3) {
    fnmac_self3<K>(a[J0], a[J0 + 1], a[J0 + 2], m);
  } else if constexpr (N == 2) {
    fnmac_self2<K>(a[J0], a[J0 + 1], m);
  } else if constexpr (N == 1) {
    fnmac_bcast<K>(a[J0], a[J0], m);
  }
}
// a[j] -= src[lane j] * m
template <int J0, int J1, typename T>
__device__ inline void fnmac_run_lanes(T (&a)[16], T src, T m) {
  constexpr int N = J1 - J0;
  if constexpr (N >= 4) {
    fnmac_lanes4<J0>(a[J0], a[J0 + 1], a[J0 + 2], a[J0 + 3], src, m);
    fnmac_run_lanes<J0 + 4, J1>(a, src, m);
  } else if constexpr (N == 3) {
    fnmac_lanes3<J0>(a[J0], a[J0 + 1], a[J0 + 2], src, m);
  } else if constexpr (N == 2) {
    fnmac_lanes2<J0>(a[J0], a[J0 + 1], src, m);
  } else if constexpr (N == 1) {
    fnmac_bcast<J0>(a[J0], src, m);
  }
}

// a[j] -= src[j][lane K] * m
template <int K, int J0, int J1, typename T>
__device__ inline void fnmac_run_each(T (&a)[16], const T (&src)[16], T m) {
  constexpr int N = J1 - J0;
  if constexpr (N >= 4) {
    fnmac_each4<K>(a[J0], a[J0 + 1], a[J0 + 2], a[J0 + 3], src[J0], src[J0 + 1], src[J0 + 2], src[J0 + 3], m);
    fnmac_run_each<K, J0 + 4, J1>(a, src, m);
  } else if constexpr (N == 3) {
    fnmac_each3<K>(a[J0], a[J0 + 1], a[J0 + 2], src[J0], src[J0 + 1], src[J0 + 2], m);
  } else if constexpr (N == 2) {
    fnmac_each2<K>(a[J0], a[J0 + 1], src[J0], src[J0 + 1], m);
  } else if constexpr (N == 1) {
    fnmac_bcast<K>(a[J0], src[J0], m);
  }
}

__device__ inline double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Reciprocal and reciprocal square root from the hardware estimate plus Newton steps (about 1 ulp;
// exact for powers of two).  They sit on the dependent chain of every pivot, where an IEEE
// division or square root would cost twice as many dependent instructions.
__device__ inline double fast_rcp(double p) {
  double r = __builtin_amdgcn_rcp(p);
  double e = __builtin_fma(-p, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-p, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ inline float fast_rcp(float p) {
  float r = __builtin_amdgcn_rcpf(p);
  const float e = __builtin_fmaf(-p, r, 1.0f);
  return __builtin_fmaf(r, e, r);
}
__device__ inline double rcp_estimate(double p) { return __builtin_amdgcn_rcp(p); }
__device__ inline float rcp_estimate(float p) { return __builtin_amdgcn_rcpf(p); }
template <typename T>
__device__ inline T rcp_refine(T p, T r) {  // one Newton step
  const T e = fma_t(-p, r, T(1));
  return fma_t(r, e, r);
}
__device__ inline double rsq_estimate(double d) { return __builtin_amdgcn_rsq(d); }
__device__ inline float rsq_estimate(float d) { return __builtin_amdgcn_rsqf(d); }
template <typename T>
__device__ inline T rsq_refine(T d, T y) {  // one Newton step towards 1/sqrt(d)
  const T t = fma_t(-d * y, y, T(1));
  return fma_t(T(0.5) * y, t, y);
}
// y ~ 1/sqrt(d) and s ~ sqrt(d)
__device__ inline void fast_rsqrt(double d, double& s, double& y) {
  y = __builtin_amdgcn_rsq(d);
  double t = __builtin_fma(-d * y, y, 1.0);
  y = __builtin_fma(0.5 * y, t, y);
  t = __builtin_fma(-d * y, y, 1.0);
  y = __builtin_fma(0.5 * y, t, y);
  s = d * y;
  s = __builtin_fma(__builtin_fma(-s, s, d), 0.5 * y, s);
}
__device__ inline void fast_rsqrt(float d, float& s, float& y) {
  y = __builtin_amdgcn_rsqf(d);
  const float t = __builtin_fmaf(-d * y, y, 1.0f);
  y = __builtin_fmaf(0.5f * y, t, y);
  s = d * y;
  s = __builtin_fmaf(__builtin_fmaf(-s, s, d), 0.5f * y, s);
}

__device__ inline double sqrt_t(double a) { return __builtin_sqrt(a); }
__device__ inline float sqrt_t(float a) { return __builtin_sqrtf(a); }

// ---- 16 x 16 register-level factorisations: lane i of a 16-lane row owns matrix row i ----

// In-place LU without pivoting of the block whose row i is a[0..15].  On exit
// a holds L (strict lower, unit diagonal implied) and U; rdiag[k] = 1/U[k][k]
// (same value in every lane).  Zero pivots are found afterwards, on U's diagonal: a test in every step
// costs as much as the step's chain (a compare, a scalar and, a select, each waiting for the last).
// Rows that do not take part in a step use a zero multiplier instead of a select.
template <typename T>
__device__ inline void lu16(T (&a)[16], T (&rdiag)[16], int i) {
  T piv = row_bcast<0>(a[0]);
  T rp = fast_rcp(piv);
  static_for<0, 16>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    rdiag[k] = rp;
    const bool below = i > k;
    const T l = below ? a[k] * rp : T(0);
    a[k] = below ? l : a[k];
    // Column k+1 first: it carries the next pivot, whose reciprocal (a chain of dependent
    // instructions) then overlaps with the independent updates of the remaining columns.
    if constexpr (k + 1 < 16) {
      fnmac_bcast<k>(a[k + 1], a[k + 1], l);
      piv = row_bcast<k + 1>(a[k + 1]);
      __builtin_amdgcn_sched_barrier(0);
      T r = rcp_estimate(piv);
      // interleave the Newton steps with the row updates, a few columns per step
      constexpr int rest = 14 - k;                 // columns k+2 .. 15
      constexpr int c1 = k + 2 + (rest + 3) / 4, c2 = k + 2 + (2 * rest + 3) / 4, c3 = k + 2 + (3 * rest + 3) / 4;
      fnmac_run_self<k, k + 2, c1>(a, l);
      __builtin_amdgcn_sched_barrier(0);
      r = rcp_refine(piv, r);
      fnmac_run_self<k, c1, c2>(a, l);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (sizeof(T) == 8) r = rcp_refine(piv, r);
      fnmac_run_self<k, c2, c3>(a, l);
      __builtin_amdgcn_sched_barrier(0);
      fnmac_run_self<k, c3, 16>(a, l);
      rp = r;
    }
  });
}

// In-place Cholesky of the block whose lower-triangle row i is a[0..i]; a[j] for j > i is
// scratch (never read for a result, may hold anything).  rdiag[k] = 1/L[k][k]; pivot[k]: its square as
// it was found, for the test d > 0 afterwards.
template <typename T>
__device__ inline void chol16(T (&a)[16], T (&rdiag)[16], T (&pivot)[16], int i) {
  T d = row_bcast<0>(a[0]);
  T s, rs;
  fast_rsqrt(d, s, rs);
  static_for<0, 16>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    pivot[k] = d;
    rdiag[k] = rs;
    const T l = (i == k) ? s : a[k] * rs;
    a[k] = (i >= k) ? l : a[k];
    // rows i <= k only touch their scratch entries a[j], j > k >= i, below.
    // Column k+1 first (next pivot), then its reciprocal square root interleaved with the rest.
    if constexpr (k + 1 < 16) {
      fnmac_bcast<k + 1>(a[k + 1], a[k], a[k]);  // a[j] -= L[i][k] * L[j][k]; L[j][k] lives in lane j
      d = row_bcast<k + 1>(a[k + 1]);
      __builtin_amdgcn_sched_barrier(0);
      T y = rsq_estimate(d);
      constexpr int rest = 14 - k;
      constexpr int c1 = k + 2 + (rest + 3) / 4, c2 = k + 2 + (2 * rest + 3) / 4, c3 = k + 2 + (3 * rest + 3) / 4;
      fnmac_run_lanes<k + 2, c1>(a, a[k], a[k]);
      __builtin_amdgcn_sched_barrier(0);
      y = rsq_refine(d, y);
      fnmac_run_lanes<c1, c2>(a, a[k], a[k]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (sizeof(T) == 8) y = rsq_refine(d, y);
      fnmac_run_lanes<c2, c3>(a, a[k], a[k]);
      __builtin_amdgcn_sched_barrier(0);
      T sq = d * y;
      sq = fma_t(fma_t(-sq, sq, d), T(0.5) * y, sq);
      fnmac_run_lanes<c3, 16>(a, a[k], a[k]);
      s = sq;
      rs = y;
    }
  });
}

// ---- a block of up to NBM columns in LDS: S[(NBM + 1)][NBM + 1], row and column NBM are dump space; rd: [NBM] reciprocals
// of the diagonal, [NBM] Cholesky's pivots ------------------------------------------------------------------------------

// A factored 16 x 16 sub-block in registers, lane i of a 16-lane row its row i, with what goes beside it.
template <typename T, int KIND>
struct DiagSub {
  T a[16], rd[16], pv[KIND == KIND_CHOL ? 16 : 1];
  __device__ __forceinline__ void factor(int lane) {
    if constexpr (KIND == KIND_LU) lu16(a, rd, lane & 15);
    else chol16(a, rd, pv, lane & 15);
  }
  // to LDS, as the sub-block at offset o (one wave)
  template <int NBM>
  __device__ __forceinline__ void store(T* const S, T* const sRd, const int lane, const int o) const {
    if (lane < 16) {
#pragma unroll
      for (int j = 0; j < 16; ++j) S[(o + lane) * (NBM + 1) + o + j] = a[j];  // (Cholesky: scratch above the diagonal, which nothing reads)
    }
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        sRd[o + j] = rd[j];
        if constexpr (KIND == KIND_CHOL) sRd[NBM + o + j] = pv[j];
      }
    }
  }
};

// The stages of a block whose first 16 x 16 sub-block is factored (bp: its size, a multiple of 16).  store(o): waves 4 .. 7
// write out the strip that begins at o, store_last(o) the one in front of the last sub-block's; inverse(upper, sub-block, unit, x): a lane's row (upper) or column of an inverse.
template <typename T, int KIND, int NBM, typename Store, typename Last, typename Inverse>
__device__ __forceinline__ void diag_stages(T* const S, T* const sRd, const int bp, const int tid, Store&& store_strip, Last&& store_last,
                                            Inverse&& inverse) {
  constexpr int NWAVES = kDiagThreads / 64, SLD = NBM + 1;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, l4 = lane >> 4;
  const int nblk = bp / kIb;
  auto factor_sub_block = [&](int o) {
    DiagSub<T, KIND> d;
#pragma unroll
    for (int j = 0; j < 16; ++j) d.a[j] = S[(o + l15) * SLD + o + j];
    d.factor(lane);
    d.template store<NBM>(S, sRd, lane, o);
  };
  // one 16 x 16 block of the inner trailing update of the stage at offset o
  auto update_block = [&](int o, int c0, int d0) {
    typename Mfma<T>::acc_t acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const T fa = -S[(c0 + l15) * SLD + o + kk * 4 + l4];
      const T fb = (KIND == KIND_LU) ? S[(o + kk * 4 + l4) * SLD + d0 + l15]
                                     : S[(d0 + l15) * SLD + o + kk * 4 + l4];
      acc = Mfma<T>::mma(fa, fb, acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15] = acc[v];
  };

  // two independent blocks at once
  auto update_block2 = [&](int o, int c0, int d0, int c1, int d1) {
    typename Mfma<T>::acc_t acc0, acc1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      acc0[v] = S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15];
      acc1[v] = S[(c1 + Mfma<T>::row_of(v, lane)) * SLD + d1 + l15];
    }
    T fa0[4], fb0[4], fa1[4], fb1[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      fa0[kk] = -S[(c0 + l15) * SLD + o + kk * 4 + l4];
      fa1[kk] = -S[(c1 + l15) * SLD + o + kk * 4 + l4];
      fb0[kk] = (KIND == KIND_LU) ? S[(o + kk * 4 + l4) * SLD + d0 + l15] : S[(d0 + l15) * SLD + o + kk * 4 + l4];
      fb1[kk] = (KIND == KIND_LU) ? S[(o + kk * 4 + l4) * SLD + d1 + l15] : S[(d1 + l15) * SLD + o + kk * 4 + l4];
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      acc0 = Mfma<T>::mma(fa0[kk], fb0[kk], acc0);
      acc1 = Mfma<T>::mma(fa1[kk], fb1[kk], acc1);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15] = acc0[v];
      S[(c1 + Mfma<T>::row_of(v, lane)) * SLD + d1 + l15] = acc1[v];
    }
  };

  // LU: blocks d, d + step, ... < nrem of one block row (row c0) of the inner trailing update, two at a time
  auto update_row = [&](int o, int c0, int d, int step, int nrem) {
    T fa[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fa[kk] = -S[(c0 + l15) * SLD + o + kk * 4 + l4];
    for (; d < nrem; d += 2 * step) {
      const bool two = d + step < nrem;  // uniform
      const int d0 = o + kIb + d * kIb, d1 = two ? d0 + step * kIb : d0;
      typename Mfma<T>::acc_t acc0, acc1;
      T fb0[4], fb1[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        acc0[v] = S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15];
        fb0[v] = S[(o + v * 4 + l4) * SLD + d0 + l15];
        acc1[v] = S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d1 + l15];
        fb1[v] = S[(o + v * 4 + l4) * SLD + d1 + l15];
      }
      if (two) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          acc0 = Mfma<T>::mma(fa[kk], fb0[kk], acc0);
          acc1 = Mfma<T>::mma(fa[kk], fb1[kk], acc1);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d1 + l15] = acc1[v];
      } else {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) acc0 = Mfma<T>::mma(fa[kk], fb0[kk], acc0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) S[(c0 + Mfma<T>::row_of(v, lane)) * SLD + d0 + l15] = acc0[v];
    }
  };
  // One 16-wide panel of the sub-block at offset o by substitution: lane t has one column (row panel: L X = P) or one row
  // (column panel: X U = P, Cholesky X L^T = P), and the 16 lanes behind the panel the identity, which becomes the
  // sub-block's inverse for the panel solves behind this block.  The sub-block is uniform over the panel, so each 16-lane
  // row keeps it in registers (lane i = its row i) and the steps take its entries as DPP broadcasts.
  auto panel = [&](auto upper_c, int o, int rem, int t) {
    constexpr bool UPPER = decltype(upper_c)::value, ROWP = KIND == KIND_LU && !UPPER;
    const int e = t < rem ? o + kIb + t : NBM;  // lanes behind the panel read and write dump space
    T f[16], rd[16], x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      f[j] = S[(o + l15) * SLD + o + j];
      if (!ROWP) rd[j] = sRd[o + j];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = ROWP ? S[(o + j) * SLD + e] : S[e * SLD + o + j];
    const int unit = t - rem;
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = unit < 0 ? x[j] : (unit == j ? T(1) : T(0));
    static_for<0, 16>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if constexpr (!ROWP) x[k] *= rd[k];
      if constexpr (UPPER) fnmac_run_each<k, k + 1, 16>(x, f, x[k]);  // U[k][j]: entry j of lane k
      else fnmac_run_lanes<k + 1, 16>(x, f[k], x[k]);                 // L[j][k]: entry k of lane j
    });
#pragma unroll
    for (int j = 0; j < 16; ++j) (ROWP ? S[(o + j) * SLD + e] : S[e * SLD + o + j]) = x[j];
    if (unit >= 0 && unit < 16) {
      inverse(upper_c, o / kIb, unit, x);
    }
  };

  // inner panels: waves 0 and 1 the row panel (Cholesky: the column panel), 2 and 3 the column panel, as far as there is one
  auto panels = [&](int o, int rem) __attribute__((always_inline)) {
    if ((wave & 1) * 64 < rem + kIb) {
      if (wave < 2) panel(std::false_type{}, o, rem, tid);
      else if constexpr (KIND == KIND_LU) panel(std::true_type{}, o, rem, tid - 128);
    }
  };
  for (int r = 0; r + 1 < nblk; ++r) {
    const int o = r * kIb;
    const int rem = bp - o - kIb;  // rows/columns to the right of / below this sub-block
    const int nrem = rem / kIb;
    // ---- inner panels; the other waves write out what is finished
    if (wave >= 4) {
      if (r > 0) store_strip(o - kIb);
    } else {
      panels(o, rem);
    }
    lds_barrier();
    // ---- inner trailing update on MFMA.  Wave 0 updates the next diagonal sub-block first and
    // factors it while the other waves update the remaining blocks (look-ahead inside the block).
    if (wave == 0) {
      update_block(o, o + kIb, o + kIb);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");  // this wave's LDS writes before its reads below
      factor_sub_block(o + kIb);
    } else if constexpr (KIND == KIND_LU) {
      // a wave stays in one block row, whose left operands it reads once; short rows are shared by several waves
      const int parts = (NWAVES - 1) / nrem, ci = (wave - 1) % nrem, part = (wave - 1) / nrem;
      if (part < parts) update_row(o, o + kIb + ci * kIb, ci == 0 && part == 0 ? parts : part, parts, nrem);
    } else {
      // q = 0 is wave 0's block; two blocks per iteration give the MFMA chains some overlap
      for (int q = wave; q < nrem * nrem; q += 2 * (NWAVES - 1)) {
        const int q2 = q + (NWAVES - 1);
        const int ci = q / nrem, di = q % nrem, ci2 = q2 / nrem, di2 = q2 % nrem;
        const bool do1 = !(KIND == KIND_CHOL && di > ci);
        const bool do2 = q2 < nrem * nrem && !(KIND == KIND_CHOL && di2 > ci2);
        if (do1 && do2) update_block2(o, o + kIb + ci * kIb, o + kIb + di * kIb, o + kIb + ci2 * kIb, o + kIb + di2 * kIb);
        else if (do1) update_block(o, o + kIb + ci * kIb, o + kIb + di * kIb);
        else if (do2) update_block(o, o + kIb + ci2 * kIb, o + kIb + di2 * kIb);
      }
    }
    lds_barrier();
  }
  // ---- the last sub-block: its inverses
  if (wave >= 4) {
    if (nblk > 1) store_last(bp - 2 * kIb);
  } else {
    panels(bp - kIb, 0);
  }
}

// --------------------------------------------------------------------------------------
template <typename T>
struct DiagArgs {
  T* A;          // top-left element of the diagonal block
  int64_t lda;
  int b;         // actual block size (<= kNbMax)
  int k0;        // global index of the block's first row/column (for info)
  int* info;     // device, may be null
  T* inv_lo;     // out: nblk inverted 16 x 16 diagonal sub-blocks of L (row-major, 256 elements each)
  T* inv_up;     // out: same for U (LU only)
  // look-ahead pipeline only (null / 0 otherwise): the block is ready once *wait_counter >= wait_target
  // (head updates finished so far); on completion *done_counter is incremented
  const int* wait_counter;
  int wait_target;
  int* done_counter;
  int* broken;   // set by a wait that gave up (see chain_wait); reported as info = -1
  long long wait_ticks;  // how long a wait may last, in ticks of the constant-rate wall clock
};

template <typename T, int KIND>
__global__ void __launch_bounds__(kDiagThreads) diag_kernel(const DiagArgs<T> g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* const S = reinterpret_cast<T*>(smem_raw);  // [kNbMax + 1][kSld]: row kNbMax and column kNbMax are dump space
  T* const sRd = S + (kNbMax + 1) * kSld;       // [kNbMax] reciprocals of the diagonal, [kNbMax] Cholesky's pivots
  constexpr int NWAVES = kDiagThreads / 64;

  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, l4 = lane >> 4;
  const int b = g.b;
  const int nblk = (b + kIb - 1) / kIb;
  const int bp = nblk * kIb;  // padded size: rows/columns b..bp-1 are identity

  if (g.wait_counter) chain_wait(g.wait_counter, g.wait_target, g.broken, g.wait_ticks, tid);
  // ---- load, padding with the identity.  Wave 0 takes the first diagonal sub-block straight to registers and
  // factors it (below) while the other waves bring the rest to LDS: a wave one row of two adjacent columns per lane,
  // all loads issued before the first LDS store.  Addresses are clamped into the block so every load is
  // unconditional (no branch, no wait between loads); out-of-block positions are replaced by the identity afterwards.
  auto load_rows = [&](auto passes) {
    constexpr int PASSES = decltype(passes)::value;
    const int c = lane * 2, r0 = wave - 1;
    T v0[PASSES], v1[PASSES];
    const int cc0 = c < b ? c : b - 1, cc1 = c + 1 < b ? c + 1 : b - 1;
#pragma unroll
    for (int it = 0; it < PASSES; ++it) {
      const int r = r0 + it * (NWAVES - 1);
      const T* p = g.A + (int64_t)(r < b ? r : b - 1) * g.lda;
      v0[it] = p[cc0];
      v1[it] = p[cc1];
    }
#pragma unroll
    for (int it = 0; it < PASSES; ++it) {
      const int r = r0 + it * (NWAVES - 1);
      if (!(r < b && c < b)) v0[it] = (r == c) ? T(1) : T(0);
      if (!(r < b && c + 1 < b)) v1[it] = (r == c + 1) ? T(1) : T(0);
    }
#pragma unroll
    for (int it = 0; it < PASSES; ++it) {
      const int r = r0 + it * (NWAVES - 1);
      if (r < bp && c < bp && (r >= kIb || c >= kIb)) {
        S[r * kSld + c] = v0[it];
        S[r * kSld + c + 1] = v1[it];
      }
    }
  };

  // Rows [o, o + 16) from column o on and columns [o, o + 16) below them are final once stage o's panels are solved.
  // Waves 4 .. 7 write them out beside the next stage's panels (Cholesky: with the zeros above the diagonal, the
  // output convention), all LDS reads first.
  auto store_strip = [&](int o) {
    const int w = wave - 4;
    constexpr int CHUNKS = kNbMax / 64, BELOW = kNbMax / kIb - 1;
    T row[4][CHUNKS], col[BELOW];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < CHUNKS; ++h) {
        const int c = o + lane + h * 64;
        row[q][h] = S[(o + w * 4 + q) * kSld + (c < kNbMax ? c : kNbMax)];
      }
#pragma unroll
    for (int q = 0; q < BELOW; ++q) {
      const int r = o + kIb + q * kIb + w * 4 + l4;
      col[q] = S[(r < kNbMax ? r : kNbMax) * kSld + o + l15];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < CHUNKS; ++h) {
        const int r = o + w * 4 + q, c = o + lane + h * 64;
        if (r < b && c < b) g.A[(int64_t)r * g.lda + c] = (KIND == KIND_LU || c <= r) ? row[q][h] : T(0);
      }
#pragma unroll
    for (int q = 0; q < BELOW; ++q) {
      const int r = o + kIb + q * kIb + w * 4 + l4;
      if (r < b) g.A[(int64_t)r * g.lda + o + l15] = col[q];
    }
  };

  if (wave == 0) {
    DiagSub<T, KIND> d;
    const T* p = g.A + (int64_t)(l15 < b ? l15 : b - 1) * g.lda;
#pragma unroll
    for (int j = 0; j < 16; ++j) d.a[j] = p[j < b ? j : b - 1];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (!(l15 < b && j < b)) d.a[j] = (l15 == j) ? T(1) : T(0);
    d.factor(lane);
    d.template store<kNbMax>(S, sRd, lane, 0);
  } else if (bp <= kNbMax / 2) {
    load_rows(std::integral_constant<int, (kNbMax / 2 + NWAVES - 2) / (NWAVES - 1)>{});
  } else {
    load_rows(std::integral_constant<int, (kNbMax + NWAVES - 2) / (NWAVES - 1)>{});
  }
  __syncthreads();

  diag_stages<T, KIND, kNbMax>(S, sRd, bp, tid, store_strip, store_strip, [&](auto upper_c, int q, int unit, const T (&x)[16]) {
    constexpr bool UPPER = decltype(upper_c)::value;
    T* const out = (UPPER ? g.inv_up : g.inv_lo) + q * 256;
#pragma unroll
    for (int j = 0; j < 16; ++j) out[UPPER ? unit * 16 + j : j * 16 + unit] = x[j];
  });

  // ---- the last sub-block; breakdown: the first pivot that is zero (LU) or not positive (Cholesky)
  if (wave >= 4) store_strip(bp - kIb);
  int info = 0;
  if (wave == 0) {
    int first = 0;
#pragma unroll
    for (int h = kNbMax / 64 - 1; h >= 0; --h) {
      const int k = h * 64 + lane;
      const T d = KIND == KIND_LU ? S[k * (kSld + 1)] : sRd[kNbMax + k];
      const unsigned long long bad = __ballot(k < b && (KIND == KIND_LU ? d == T(0) : !(d > T(0))));
      if (bad) first = h * 64 + __builtin_ctzll(bad) + 1;
    }
    info = first ? g.k0 + first : 0;
  }
  if (tid == 0 && g.info) {
    if (g.k0 == 0) *g.info = info;  // first block of the call: initialise
    else if (info != 0 && *g.info == 0) *g.info = info;
    if (g.broken && __hip_atomic_load(g.broken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) *g.info = -1;
  }
  if (g.done_counter) chain_signal(g.done_counter, 1, tid);
}

template <typename T>
constexpr int diag_lds_bytes() {
  return ((kNbMax + 1) * kSld + 2 * kNbMax) * (int)sizeof(T);
}

// Zero a few ints (the hand-over counters) with a kernel: usable under stream capture, unlike a memset node.
static __global__ void zero_ints_kernel(int* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// One wave that waits in place until a hand-over counter reaches its target (bounded like every such wait): put in
// front of a kernel on a stream that would otherwise wait for another stream's event.
static __global__ void gate_kernel(const int* counter, int target, int* broken, long long wait_ticks) {
  chain_wait(counter, target, broken, wait_ticks, (int)threadIdx.x);
}

// A 16 x 16 identity and three zeroed counters (the hand-over self-test's input).
static __global__ void identity16_kernel(double* a, int* counters) {
  const int t = (int)threadIdx.x;
  a[t] = (t / 16 == t % 16) ? 1.0 : 0.0;
  if (t < 3) counters[t] = 0;
}

// Zero the strict upper triangle (Cholesky output convention).  nb = 1: all of it.  nb > 1: only the
// blocks above the block diagonal of width nb, which no kernel of the factorisation touches, so that
// this can run beside the first steps; the diagonal-block kernel zeroes its own block's upper part.
template <typename T>
__global__ void __launch_bounds__(256) zero_upper_kernel(T* A, int64_t lda, int n, int nb) {
  const int col = (int)blockIdx.x * 256 + (int)threadIdx.x;
  for (int row = (int)blockIdx.y; row < n; row += (int)gridDim.y)
    if (col >= (row / nb + 1) * nb && col < n) A[(int64_t)row * lda + col] = T(0);
}

}  // namespace dla
