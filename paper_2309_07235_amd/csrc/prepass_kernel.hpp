// What a solve prepares from the factor alone, behind the inverses of the 128-row diagonal blocks (tri_prepare_kernel):
//   pair_kernel       the off-diagonal quarter that makes two of them the inverse of a 256-row block,
//   look_back_kernel  the products M of the inverses with the factor's blocks beside them,
// each one launch for both passes.  With the negated inverses N = -W:
//   inv [ L1 0; L21 L2 ]:  N21 = N2 (L21 N1)        inv [ U1 U12; 0 U2 ]:  N12 = N1 (U12 N2)
//   M_i = -N_i [L_{i,i-2}, L_{i,i-1}]  (forward)    M_k = -N_k [U_{k,k+1}, U_{k,k+2}]  (backward; Cholesky: its transpose)
// What bounds them is latency: a launch is 10 - 30 us for 0.1 - 1 GFLOP.  So nothing is cleared first (a plain product is
// stored, not subtracted from zero), both products of a quarter stay in one workgroup, and the zero halves of triangular
// operands are left out.  Prepare calls in us, fill, inverses, one or two grouped GEMM launches per product and pass against
// this: LU fp64 n = 300 59 -> 37, n = 1000 72 -> 42, n = 4000 106 -> 63, n = 8192 188 -> 95; Cholesky n = 4000 93 -> 62; fp32 LU
// n = 4000 79 -> 44.  k-slabs of 256 or 512 bytes in the products M: no faster at any size, 512 slower from n = 2000 on.
#pragma once
#include "trisolve_kernel.hpp"
#include "gemm_wide_kernel.hpp"

namespace dla {

template <typename T>
struct PrepassArgs {
  const T* F;
  int64_t lda;
  int n;
  T* wf;   // negated inverses, forward pass: one 256 x 256 area per block
  T* wb;   // and backward pass (LU)
  T* mf;   // M of the forward pass: 256 x 512 each
  T* mb;   // M of the backward pass (Cholesky: its transpose, 512 x 256)
};

// ---- pairing.  One workgroup per 16 columns of a quarter; its columns need nothing of the others.  A wave owns 16 rows of
// both products; the first one's result goes through LDS.
constexpr int kPairThreads = 512;
constexpr int kPairSlices = kNbMax / 16;
static_assert(kPairThreads / 64 * 16 == kNbMax, "a wave per 16 rows");
// of one pass: the slices of a block go to one XCD, whose L2 then serves the operands that they share
__host__ __device__ inline int pair_workgroups(int n) {
  const int blocks = (n + kTriPair - 1) / kTriPair;
  return (blocks + kNumXcd - 1) / kNumXcd * kNumXcd * kPairSlices;
}

template <typename T, int KIND>
__global__ void __launch_bounds__(kPairThreads) pair_kernel(const PrepassArgs<T> g) {
  using acc_t = typename Mfma<T>::acc_t;
  using R2 = typename WideRun<T, 2>::type;
  constexpr int STEPS = kNbMax / 4;       // k-steps; k of step s: 8 (s / 2) + 2 l4 + s % 2
  constexpr int64_t LW = kTriPair;
  __shared__ T ts[kNbMax * 17];
  const int blocks = (g.n + kTriPair - 1) / kTriPair, per_pass = pair_workgroups(g.n);
  int bid = (int)blockIdx.x;
  const bool back = bid >= per_pass;
  if (back) bid -= per_pass;
  const int p = bid % kNumXcd + bid / (kNumXcd * kPairSlices) * kNumXcd, slice = bid / kNumXcd % kPairSlices, k0 = p * kTriPair;
  if (p >= blocks) return;  // uniform
  const int b2 = g.n - k0 - kNbMax < kNbMax ? g.n - k0 - kNbMax : kNbMax;
  if (b2 <= 0) return;  // uniform: a last block without a partner
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, l4 = lane >> 4;
  T* const W = (back ? g.wb : g.wf) + (int64_t)p * LW * LW;
  const T* const A = back ? g.F + (int64_t)k0 * g.lda + k0 + kNbMax : g.F + (int64_t)(k0 + kNbMax) * g.lda + k0;
  T* const W2 = W + kNbMax * LW + kNbMax;
  const T* const P1 = back ? W2 : W;  // right operand of the first product
  const T* const P2 = back ? W : W2;  // left operand of the second one
  const int rows = back ? kNbMax : b2, depth = back ? b2 : kNbMax, cols = back ? b2 : kNbMax;  // of A; of the quarter
  T* const Q = back ? W + kNbMax : W + kNbMax * LW;
  // the other quarter is zero
  {
    T* const Z = back ? W + kNbMax * LW : W + kNbMax;
    const int zrows = back ? b2 : kNbMax;
    for (int r = tid >> 4; r < zrows; r += kPairThreads / 16) Z[r * LW + slice * 16 + (tid & 15)] = T(0);
  }
  const int c = slice * 16 + l15;
  if (slice * 16 >= cols) return;  // uniform
  const int r0 = wave * 16, row = r0 + l15;
  const T* const Ar = A + (int64_t)(row < rows ? row : rows - 1) * g.lda;
  const T* const Pr = P2 + (int64_t)(row < rows ? row : rows - 1) * LW;
  const T* const Pc = P1 + (c < cols ? c : cols - 1);
  T a[STEPS], b[STEPS], w[STEPS];
  auto k_of = [&](int s) { return 8 * (s >> 1) + 2 * l4 + (s & 1); };
  // left operands as pairs (16 bytes in fp64, aligned to an element); a depth that is not whole: element by element, zero beyond
  auto load_left = [&](T (&x)[STEPS], const T* q, int kc) __attribute__((always_inline)) {
    if (kc == kNbMax) {  // uniform
#pragma unroll
      for (int s = 0; s < STEPS; s += 2) {
        const R2 v = *reinterpret_cast<const R2*>(q + k_of(s));
        x[s] = v[0];
        x[s + 1] = v[1];
      }
    } else {
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
        const T v = q[k_of(s) < kc ? k_of(s) : kc - 1];
        x[s] = k_of(s) < kc ? v : T(0);
      }
    }
  };
  load_left(a, Ar, depth);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int k = k_of(s);
    const T v = Pc[(k < depth ? k : depth - 1) * LW];
    b[s] = k < depth ? v : T(0);
  }
  load_left(w, Pr, rows);
  // P1's column block `slice` is zero above (forward: lower triangular) or below (upper) its diagonal, P2's row block likewise
  acc_t acc = {0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < STEPS; s += 4)
    if (back ? s / 4 <= slice : s / 4 >= slice) {  // uniform
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = Mfma<T>::mma(a[s + e], b[s + e], acc);
    }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = r0 + Mfma<T>::row_of(v, lane);
    ts[r * 17 + l15] = r < rows ? acc[v] : T(0);
  }
  lds_barrier();
  acc = acc_t{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < STEPS; s += 4)
    if (back ? s / 4 >= wave : s / 4 <= wave) {  // uniform
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = Mfma<T>::mma(w[s + e], ts[k_of(s + e) * 17 + l15], acc);
    }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = r0 + Mfma<T>::row_of(v, lane);
    if (r < rows && c < cols) Q[r * LW + c] = acc[v];
  }
}

// ---- the products M, 64 x 64 tiles of gemm_wide_tile.  A block's tiles go to one XCD, whose L2 then holds its operands.
constexpr int kLookTile = 64, kLookThreads = 512;
constexpr int kLookTiles = kTriPair / kLookTile * (2 * kTriPair / kLookTile);
template <typename T>
using LookShape = WideShape<T, 4, 2, 1, 2, 128 / (int)sizeof(T), false>;

inline int look_back_workgroups(int64_t n) {
  const int problems = 2 * (int)((n + kTriPair - 1) / kTriPair - 1);
  return (problems + kNumXcd - 1) / kNumXcd * kNumXcd * kLookTiles;
}

template <typename T, int KIND, typename Off>
__global__ void __launch_bounds__(kLookThreads) look_back_kernel(const PrepassArgs<T> g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int64_t SB = kTriPair;
  const int last = (g.n + kTriPair - 1) / kTriPair - 1;
  const int bid = (int)blockIdx.x, q = bid % kNumXcd + bid / kNumXcd / kLookTiles * kNumXcd, tile = bid / kNumXcd % kLookTiles;
  if (q >= 2 * last) return;  // uniform
  const bool back = q >= last;
  const int i = back ? q - last : q + 1;  // block row
  auto rows_of = [&](int j) { return g.n - j * kTriPair < kTriPair ? g.n - j * kTriPair : kTriPair; };
  GemmProblem<T> P;
  P.C2 = nullptr;
  P.ldc2 = 0;
  P.K = rows_of(i);
  int ti, tj;
  if (KIND == KIND_CHOL && back) {  // [L_{i+1,i}; L_{i+2,i}] W_i, W_i lower triangular
    ti = tile / (kTriPair / kLookTile);
    tj = tile % (kTriPair / kLookTile);
    const int64_t c0 = (int64_t)(i + 1) * SB;
    const int skip = tj * kLookTile;
    P.A = g.F + c0 * g.lda + i * SB + skip;
    P.lda = g.lda;
    P.B = g.wf + (int64_t)i * SB * SB + skip * SB;
    P.ldb = SB;
    P.C = g.mb + (int64_t)i * 2 * SB * SB;
    P.ldc = SB;
    P.M = (int)(g.n - c0 < 2 * SB ? g.n - c0 : 2 * SB);
    P.N = kTriPair;
    P.K -= skip;
  } else {
    ti = tile / (2 * kTriPair / kLookTile);
    tj = tile % (2 * kTriPair / kLookTile);
    const int64_t c0 = (back ? i + 1 : i >= 2 ? i - 2 : 0) * SB;
    const int skip = back ? ti * kLookTile : 0;  // W_i upper triangular: nothing in front of the tile's rows
    P.A = (back ? g.wb : g.wf) + (int64_t)i * SB * SB + skip;
    P.lda = SB;
    P.B = g.F + (i * SB + skip) * g.lda + c0;
    P.ldb = g.lda;
    P.C = (back ? g.mb : g.mf) + (int64_t)i * 2 * SB * SB;
    P.ldc = 2 * SB;
    P.M = P.K;
    P.N = (int)(back ? (g.n - c0 < 2 * SB ? g.n - c0 : 2 * SB) : i * SB - c0);
    if (back) P.K -= skip;
    else if (P.K > (ti + 1) * kLookTile) P.K = (ti + 1) * kLookTile;  // lower triangular: nothing behind them
  }
  if (ti * kLookTile >= P.M || tj * kLookTile >= P.N) return;  // uniform
  gemm_wide_tile<T, 4, 2, 1, 2, 128 / (int)sizeof(T), OP_NEGATE, Off>(P, ti, tj, reinterpret_cast<T*>(smem_raw));
}

}  // namespace dla
