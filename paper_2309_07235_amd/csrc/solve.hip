// Host driver of the solves with the factors: A X = B as  L Y = B, U X = Y  (LU) or
// L Y = B, L^T X = Y  (Cholesky), B overwritten by X.  Blocked substitution over row blocks of up
// to 256.  A pre-pass, independent of B, inverts every diagonal block: the 128-row blocks by
// tri_prepare_kernel, then pairs of them joined into the inverse of a 256-row block,
//   inv [ L1  0  ] = [  W1        0  ]        inv [ U1 U12 ] = [ V1  -V1 U12 V2 ]
//       [ L21 L2 ]   [ -W2 L21 W1  W2 ]            [ 0  U2  ]   [ 0    V2       ]
// (pair_kernel), then the products M below (look_back_kernel): three launches.
//
// The chain of the substitution is latency bound (every step waits for the one before it), so a
// block step is ONE grouped launch (or, with few right-hand sides, one hop inside a launch).  With W_i the inverse of diagonal block i, the plain step
//   X_i = W_i (B_i - sum_{j<i} L_ij X_j)
// is split as  X_i = Z_i - M_i [X_{i-2}; X_{i-1}],  Z_i = W_i (B_i - sum_{j<i-2} L_ij X_j),
// M_i = W_i [L_{i,i-2}, L_{i,i-1}]  (the pre-pass forms M_i, one product per block).  The launch that
// follows X_k then carries three products that read nothing newer than X_k:
//   (a) X_{k+1} = Z_{k+1} - M_{k+1} [X_{k-1}; X_k]
//   (b) Z_{k+2} = W_{k+2} B_{k+2}            (B_{k+2} already holds the contributions of X_0..X_{k-1})
//   (c) B_i -= L_ik X_k  for the blocks i >= k + 3
// and the backward pass mirrors it from the last block upwards.  A launch has one operation for all
// its products, the subtracting one, so the pre-pass stores the NEGATED inverses N = -W and every
// product is  C -= A * B  on a target that starts at zero where a plain product is meant
// (Z = 0 - N B,  M = 0 - N L).  For Cholesky the backward inverse is the transpose of the forward one
// and the backward pass reads N, M^T and L's block rows as transposed left operands, so it needs no
// inverses of its own.  The forward pass leaves Y in the workspace and spoils B; the backward pass
// builds X in a second workspace area and stores each finished block to B as well.
// Up to 64 right-hand sides both passes are one launch of flow_kernel, whose workgroups wait for each other; above that the
// chain's launches run on skinny_kernel up to 128 right-hand sides (256 of a small system) and on gemm_wide_kernel beyond.
// The pre-pass and the two passes can be called separately (one pre-pass, many solves with its workspace).
#include "prepass_kernel.hpp"
#include "skinny_kernel.hpp"
#include "flow_kernel.hpp"
#include "host_common.hpp"

namespace dla {

template <typename T, int MODE>
static int launch_prepare(const TriPrepareArgs<T>& a, const FlowInit<T>& init, hipStream_t st) {
  auto kern = tri_prepare_kernel<T, MODE>;
  static LdsLimitOnce lds_limit;
  if (!lds_limit.ensure(reinterpret_cast<const void*>(kern), trisolve_lds_bytes<T>())) return DLA_ERR_HIP;
  const int grid = kTriHalves * (int)((a.n + kNbMax - 1) / kNbMax);
  ProfileScope scope(PHASE_TRSM, 0.0, st);
  hipLaunchKernelGGL(kern, dim3((unsigned)(grid + flow_init_workgroups(init))), dim3(kTriThreads), trisolve_lds_bytes<T>(), st, a, init);
  return launch_status(__func__);
}

template <typename T, int MODE_A, int MODE_B>
static int launch_prepare_both(const TriPrepareArgs<T>& a, const TriPrepareArgs<T>& b, const FlowInit<T>& init, hipStream_t st) {
  auto kern = tri_prepare_both_kernel<T, MODE_A, MODE_B>;
  static LdsLimitOnce lds_limit;
  if (!lds_limit.ensure(reinterpret_cast<const void*>(kern), trisolve_lds_bytes<T>())) return DLA_ERR_HIP;
  const int grid = 2 * kTriHalves * (int)((a.n + kNbMax - 1) / kNbMax);
  ProfileScope scope(PHASE_TRSM, 0.0, st);
  hipLaunchKernelGGL(kern, dim3((unsigned)(grid + flow_init_workgroups(init))), dim3(kTriThreads), trisolve_lds_bytes<T>(), st, a, b, init);
  return launch_status(__func__);
}

template <typename T>
static int launch_skinny(bool at, const SkinnyGroup<T>& g, int workgroups, int kmax, double flops, hipStream_t st) {
  ProfileScope scope(PHASE_GEMM, flops, st);
  const dim3 grid((unsigned)workgroups), block(kSkinnyThreads);
  if (kmax <= 256) {
    if (at) hipLaunchKernelGGL((skinny_kernel<T, true, 16>), grid, block, 0, st, g);
    else hipLaunchKernelGGL((skinny_kernel<T, false, 16>), grid, block, 0, st, g);
  } else {
    if (at) hipLaunchKernelGGL((skinny_kernel<T, true, 32>), grid, block, 0, st, g);
    else hipLaunchKernelGGL((skinny_kernel<T, false, 32>), grid, block, 0, st, g);
  }
  return launch_status(__func__);
}

template <typename T, int KIND>
static int launch_flow(const FlowArgs<T>& a, int nb, double flops, hipStream_t st) {
  ProfileScope scope(PHASE_GEMM, flops, st);
  const dim3 grid((unsigned)flow_pieces(a.blocks, a.tiles_n)), block(kFlowThreads);
  if (nb == 1) hipLaunchKernelGGL((flow_kernel<T, KIND, 1>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((flow_kernel<T, KIND, 2>), grid, block, 0, st, a);
  return launch_status(__func__);
}

template <typename T>
__global__ void solve_zero_kernel(T* p, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = T(0);
}

// Workspace, in elements: per 256-row block a 256 x 256 negated inverse for the forward and one for the
// backward pass (LU), 128 x 128 for each (flow_kernel's S, up to 64 right-hand sides), and a 256 x 512 area M for each
// pass (the first one of the forward pass, which has none, for flow_kernel's flags); then the n x nrhs areas Y and X (leading dimension nrhs rounded up to even), which
// a call sets to zero, or to what flow_kernel never publishes, before its passes.
static int64_t pairs_of(int64_t n) { return (n + kTriPair - 1) / kTriPair; }
static int64_t block_elems(int64_t n) {
  return 2 * pairs_of(n) * ((int64_t)kTriPair * kTriPair + (int64_t)kNbMax * kNbMax + 2 * (int64_t)kTriPair * kTriPair);
}
static int64_t y_ld(int64_t nrhs) { return (nrhs + 1) / 2 * 2; }
size_t solve_workspace_bytes_impl(int64_t n, int64_t nrhs, dla_dtype dt) {
  return ((size_t)block_elems(n) + 2 * (size_t)n * (size_t)y_ld(nrhs)) * (dt == DLA_F64 ? 8 : 4);
}

// The products of the chain with many right-hand sides take gemm_wide_kernel, whose launch
// picks the tile: N = 8192 with 1024 right-hand sides, fp32, 2.79 -> 2.18 ms against 32 x 32 tiles of gemm_kernel.  This
// schedule is for what that kernel does not take (leading dimensions beyond its offsets, fp32 systems of up to 32 rows).
static const GemmSchedule kSolveTiles = {32, 32, 16, 4, 16, 16};
template <typename T>
static int launch_products(int op, GemmGroup<T>& g, int np, int tiles, double flops, hipStream_t st) {
  for (int q = np; q < kMaxGroup; ++q) g.prob[q] = g.prob[0];
  g.nprob = np;
  g.total_tiles = tiles;
  ProfileScope scope(PHASE_GEMM, flops, st);
  return gemm_wide_takes<T>(op, g) ? launch_gemm_wide<T>(op, g, st) : launch_gemm<T>(kSolveTiles, op, g, st);
}

template <typename T, int KIND>
static int launch_pairing(const PrepassArgs<T>& a, hipStream_t st) {
  if (a.n <= kNbMax) return DLA_SUCCESS;
  ProfileScope scope(PHASE_GEMM, 0.0, st);
  hipLaunchKernelGGL((pair_kernel<T, KIND>), dim3((unsigned)((KIND == KIND_LU ? 2 : 1) * pair_workgroups(a.n))), dim3(kPairThreads), 0, st, a);
  return launch_status(__func__);
}

template <typename T, int KIND, typename Off>
static int launch_look_back_as(const PrepassArgs<T>& a, hipStream_t st) {
  auto kern = look_back_kernel<T, KIND, Off>;
  using S = LookShape<T>;
  static_assert(S::NT == kLookThreads, "threads");
  static LdsLimitOnce lds_limit;
  if (!lds_limit.ensure(reinterpret_cast<const void*>(kern), S::BYTES)) return DLA_ERR_HIP;
  ProfileScope scope(PHASE_GEMM, 0.0, st);
  hipLaunchKernelGGL(kern, dim3((unsigned)look_back_workgroups(a.n)), dim3(kLookThreads), S::BYTES, st, a);
  return launch_status(__func__);
}
template <typename T, int KIND>
static int launch_look_back(const PrepassArgs<T>& a, hipStream_t st) {
  if (a.n <= kTriPair) return DLA_SUCCESS;
  if (a.lda > (1 << 24)) return launch_look_back_as<T, KIND, uint64_t>(a, st);  // beyond 32-bit element offsets inside a tile
  return launch_look_back_as<T, KIND, uint32_t>(a, st);
}

// phases: kSolvePrepare = the pre-pass (independent of B; leaves the negated inverses and M in the workspace),
// kSolveApply = the two passes over B with a workspace the pre-pass has filled for this factor; both = a whole solve.
template <typename T, int KIND>
int solve_impl(const T* F, int64_t n, int64_t lda, T* B, int64_t nrhs, int64_t ldb, void* ws, size_t ws_bytes,
               hipStream_t st, int phases, FlowWaits waits) {
  const bool prepare = phases & kSolvePrepare, apply = (phases & kSolveApply) && nrhs > 0;
  if (n == 0 || (nrhs == 0 && (phases & kSolveApply))) return DLA_SUCCESS;
  const dla_dtype dt = sizeof(T) == 8 ? DLA_F64 : DLA_F32;
  if (!ws || ws_bytes < solve_workspace_bytes_impl(n, nrhs, dt) || ((uintptr_t)ws % 256)) return DLA_ERR_WORKSPACE;
  constexpr int BOP = (KIND == KIND_LU) ? OP_SUB : OP_SUB_TN;  // the backward pass's one operation
  const int64_t nb = kNbMax, sb = kTriPair;
  const int64_t pairs = pairs_of(n);
  const int nblk = (int)pairs, last = nblk - 1;
  T* const wf = static_cast<T*>(ws);      // negated inverses, forward pass: pairs x (256 x 256)
  T* const wb = wf + pairs * sb * sb;     // negated inverses, backward pass (LU)
  T* const tf = wb + pairs * sb * sb;     // S of flow_kernel: 2 x pairs x (128 x 128)
  T* const mf = tf + 2 * pairs * nb * nb; // M of the forward pass: pairs x (256 x 512)
  T* const mb = mf + pairs * sb * 2 * sb; // M of the backward pass (Cholesky: its transpose, 512 x 256)
  T* const Y = mb + pairs * sb * 2 * sb;  // n x nrhs: Z and then the solution of the forward pass
  static_assert(kFlowBlock == kTriPair, "both passes' blocks are the pre-pass's");
  const int64_t ldy = y_ld(nrhs);
  T* const X = Y + n * ldy;               // n x nrhs: Z and then the solution of the backward pass
  auto rows_of = [&](int i) { return n - (int64_t)i * sb < sb ? n - (int64_t)i * sb : sb; };
  auto Nf = [&](int i) { return wf + (int64_t)i * sb * sb; };
  auto Nb = [&](int i) { return wb + (int64_t)i * sb * sb; };
  int rc;
  // Few right-hand sides: both passes in one launch (flow_kernel).  64 is where the two areas for S end to fit in their
  // part of the workspace; the line lies there and not below because one launch is faster all the way (a prepared LU solve, fp64, us,
  // launches against this, 1 / 16 / 64 right-hand sides: n = 300 23 / 23 / 24 against 15 / 15 / 16, n = 1000 46 / 47 / 51
  // against 26 / 26 / 33, n = 2000 102 / 103 / 110 against 48 / 50 / 72, n = 4000 211 / 212 / 255 against 102 / 108 / 186,
  // n = 8192 571 / 578 / 746 against 271 / 283 / 566; fp32 n = 4000 182 / 180 / 204 against 86 / 96 / 155).  A workgroup takes
  // two column blocks where one each would be more workgroups than fit beside each other by much (one against two, n = 2000 with 32
  // 61 / 73, with 64 72 / 83; n = 4000 with 32 141 / 143, with 64 199 / 186; n = 8192 with 32 419 / 367, with 64 672 / 566).
  const int flow_nb = nrhs > 16 && n * nrhs > 128000 ? 2 : 1;
  const int tiles_n = (int)((nrhs + 16 * flow_nb - 1) / (16 * flow_nb));
  // (its flags and claims lie in the first block's M, room for 683 blocks in fp32 with two column tiles, n = 174 848; beyond: launches)
  const bool flow = nrhs <= 64 && lda <= kFlowMaxLd && flow_ints(nblk, tiles_n) * (int64_t)sizeof(int) <= 2 * sb * sb * (int64_t)sizeof(T);
  int* const ints = reinterpret_cast<int*>(mf);  // (the first block has no M)
  FlowInit<T> init{Y, nblk > kFlowLook + 1 ? tf : nullptr, 0, ints, 0};  // S: where the pre-pass keeps nothing
  if (apply && flow) {
    init.count = 2 * n * ldy;
    init.nints = (int)flow_ints(nblk, tiles_n);
  }
  if (prepare) {
    if (KIND == KIND_LU)
      rc = launch_prepare_both<T, TRI_LOWER_UNIT, TRI_UPPER>(TriPrepareArgs<T>{F, lda, n, wf, T(-1)}, TriPrepareArgs<T>{F, lda, n, wb, T(-1)}, init, st);
    else
      rc = launch_prepare<T, TRI_LOWER>(TriPrepareArgs<T>{F, lda, n, wf, T(-1)}, init, st);
    if (rc != DLA_SUCCESS) return rc;
    const PrepassArgs<T> pa{F, lda, (int)n, wf, wb, mf, mb};
    if ((rc = launch_pairing<T, KIND>(pa, st)) != DLA_SUCCESS || (rc = launch_look_back<T, KIND>(pa, st)) != DLA_SUCCESS) return rc;
  }
  if (!apply) return DLA_SUCCESS;
  if (flow) {
    if (!prepare) {
      hipLaunchKernelGGL(flow_init_kernel<T>, dim3((unsigned)flow_init_workgroups(init)), dim3(kFlowThreads), 0, st, init);
      if (launch_status(__func__) != DLA_SUCCESS) return DLA_ERR_HIP;
    }
    int* const done = ints + 2 * nblk * tiles_n * kFlowTiles;
    FlowArgs<T> a{F, B, wf, KIND == KIND_LU ? wb : wf, mf, mb, Y, X, tf, ints, done, done + tiles_n + 1,
                  waits == FlowWaits::kGiveUp ? 0 : kFlowWaitTicks, waits == FlowWaits::kOrdinary ? kFlowSearchTicks : waits == FlowWaits::kAbsent ? 2000 : 0,
                  waits == FlowWaits::kAbsent ? 3 : -1,
                  lda, ldb, ldy, (int)n, (int)nrhs, nblk, tiles_n, flow_expected((int)n, nblk)};
    return launch_flow<T, KIND>(a, flow_nb, 2.0 * (double)n * (double)n * (double)nrhs, st);
  }
  // ---- the targets of the passes' subtracting products that stand for plain ones start at zero
  {
    const int64_t count = 2 * n * ldy;
    hipLaunchKernelGGL(solve_zero_kernel<T>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, Y, count);
    if (launch_status(__func__) != DLA_SUCCESS) return DLA_ERR_HIP;
  }
  // ---- the chain: one grouped launch per block step
  struct Part {
    const T *a, *b;
    T *c, *c2;
    int64_t la, lb, lc, lc2, M, K;
    int many;  // 1 for product (c): many blocks, the factor as its left operand
  };
  // While a launch of the chain is a few hundred to a few thousand 16 x 16 blocks, what matters is how soon its
  // longest product ends: the skinny kernel (one block per workgroup, k split over its waves).  With more work per launch
  // the tiled GEMM's reuse wins.  The two passes of a prepared LU solve, fp64, skinny against tiled: N = 1000 with 256
  // right-hand sides 66 against 87 us; N = 4000 with 64 251 against 356, 128 331 against 417, 256 490 against 505, 320
  // 0.93 of the skinny time; N = 8192 with 128 1085 against 1194, 160 0.98, 256 0.85.  fp32 crosses a little earlier
  // (N = 4000, 256: 0.91; N = 8192, 128: 1.00), Cholesky where LU does.
  const bool skinny = nrhs <= 128 || (nrhs <= 256 && n * nrhs <= 1200000);
  static_assert(2 * kTriPair <= kSkinnyMaxK, "the look-back product's depth");
  auto launch_parts = [&](int op, const Part* parts, int count) -> int {
    if (skinny) {
      SkinnyGroup<T> sg;
      int np = 0, wgs = 0, kmax = 0;
      double flops = 0.0;
      for (int q = 0; q < count; ++q) {
        const Part& P = parts[q];
        if (P.M <= 0 || P.K <= 0) continue;
        SkinnyPart<T>& sp = sg.part[np++];
        const int wide = (P.many && nrhs > 16 && P.K <= 256) ? 1 : 0;
        sp = SkinnyPart<T>{P.a, P.b, P.c, P.c2, P.la, P.lb, P.lc, P.lc2, (int)P.M, (int)nrhs, (int)P.K,
                           (int)((nrhs + (wide ? 31 : 15)) / (wide ? 32 : 16)), wgs, wide};
        wgs += skinny_workgroups(P.M, sp.tiles_n);
        kmax = P.K > kmax ? (int)P.K : kmax;
        flops += 2.0 * (double)P.M * (double)nrhs * (double)P.K;
      }
      if (np == 0) return DLA_SUCCESS;
      for (int q = np; q < kSkinnyMaxParts; ++q) sg.part[q] = sg.part[0];
      sg.nparts = np;
      return launch_skinny<T>(op == OP_SUB_TN, sg, wgs, kmax, flops, st);
    }
    GemmGroup<T> g;
    int np = 0, tiles = 0;
    double flops = 0.0;
    for (int q = 0; q < count; ++q) {
      const Part& P = parts[q];
      if (P.M <= 0 || P.K <= 0) continue;
      g.prob[np] = make_problem<T>(kSolveTiles, op, P.a, P.la, P.b, P.lb, P.c, P.lc, P.M, nrhs, P.K, tiles);
      g.prob[np].C2 = P.c2;
      g.prob[np].ldc2 = P.lc2;
      tiles += problem_tiles(kSolveTiles, op, g.prob[np]);
      flops += 2.0 * (double)P.M * (double)nrhs * (double)P.K;
      ++np;
    }
    return np == 0 ? (int)DLA_SUCCESS : launch_products<T>(op, g, np, tiles, flops, st);
  };
  // ---- forward.  Z_i and then Y_i live in rows i of Y; B is updated in place (part c).
  {
    Part head[2] = {{Nf(0), B, Y, nullptr, sb, ldb, ldy, 0, rows_of(0), rows_of(0)}, {}};
    if (nblk > 1) head[1] = Part{Nf(1), B + sb * ldb, Y + sb * ldy, nullptr, sb, ldb, ldy, 0, rows_of(1), rows_of(1)};
    if ((rc = launch_parts(OP_SUB, head, 2)) != DLA_SUCCESS) return rc;
  }
  for (int k = 0; k < last; ++k) {
    const int64_t k0 = (int64_t)k * sb;
    const int64_t c0 = (int64_t)(k >= 1 ? k - 1 : 0) * sb, kc = k0 + sb - c0;  // rows of Y that M_{k+1} multiplies
    const int64_t r3 = k0 + 3 * sb;                                            // first row of part (c)
    // (c) first: its workgroups wait longest for their operand (the factor, from HBM), so they are dispatched
    // first (N = 4000, 64 right-hand sides: 0.365 ms against 0.380 ms with (c) last)
    Part parts[3] = {
        {},
        {mf + (int64_t)(k + 1) * sb * 2 * sb, Y + c0 * ldy, Y + (k0 + sb) * ldy, nullptr, 2 * sb, ldy, ldy, 0, rows_of(k + 1), kc, 0},
        {}};
    if (r3 < n) parts[0] = Part{F + r3 * lda + k0, Y + k0 * ldy, B + r3 * ldb, nullptr, lda, ldy, ldb, 0, n - r3, sb, 1};
    if (k + 2 < nblk)
      parts[2] = Part{Nf(k + 2), B + (k0 + 2 * sb) * ldb, Y + (k0 + 2 * sb) * ldy, nullptr, sb, ldb, ldy, 0, rows_of(k + 2), rows_of(k + 2), 0};
    if ((rc = launch_parts(OP_SUB, parts, 3)) != DLA_SUCCESS) return rc;
  }
  // ---- backward.  Z_k and then X_k live in rows k of X (finished blocks are stored to B as well); Y is
  // updated in place (part c).  Cholesky: every left operand is read transposed (stored k x m).
  {
    const int64_t l0 = (int64_t)last * sb;
    Part head[2] = {{KIND == KIND_LU ? Nb(last) : Nf(last), Y + l0 * ldy, X + l0 * ldy, B + l0 * ldb, sb, ldy, ldy, ldb,
                     rows_of(last), rows_of(last)},
                    {}};
    if (last >= 1)
      head[1] = Part{KIND == KIND_LU ? Nb(last - 1) : Nf(last - 1), Y + (l0 - sb) * ldy, X + (l0 - sb) * ldy, nullptr, sb, ldy, ldy, 0, sb, sb};
    if ((rc = launch_parts(BOP, head, 2)) != DLA_SUCCESS) return rc;
  }
  for (int k = last; k >= 1; --k) {
    const int64_t k0 = (int64_t)k * sb;
    const int64_t kc = (n < k0 + 2 * sb ? n : k0 + 2 * sb) - k0;  // rows of X that M_{k-1} multiplies: blocks k, k+1
    const int64_t r1 = k0 - 2 * sb;                               // part (c) covers rows 0 .. r1
    const T* const m_prev = mb + (int64_t)(k - 1) * sb * 2 * sb;
    Part parts[3] = {
        {},
        {m_prev, X + k0 * ldy, X + (k0 - sb) * ldy, B + (k0 - sb) * ldb, KIND == KIND_LU ? 2 * sb : sb, ldy, ldy, ldb, sb, kc, 0},
        {}};
    if (r1 > 0) parts[0] = Part{KIND == KIND_LU ? F + k0 : F + k0 * lda, X + k0 * ldy, Y, nullptr, lda, ldy, ldy, 0, r1, rows_of(k), 1};
    if (k >= 2)
      parts[2] = Part{KIND == KIND_LU ? Nb(k - 2) : Nf(k - 2), Y + (k0 - 2 * sb) * ldy, X + (k0 - 2 * sb) * ldy, nullptr, sb, ldy, ldy, 0, sb, sb, 0};
    if ((rc = launch_parts(BOP, parts, 3)) != DLA_SUCCESS) return rc;
  }
  return DLA_SUCCESS;
}

template int solve_impl<double, KIND_LU>(const double*, int64_t, int64_t, double*, int64_t, int64_t, void*, size_t, hipStream_t, int, FlowWaits);
template int solve_impl<float, KIND_LU>(const float*, int64_t, int64_t, float*, int64_t, int64_t, void*, size_t, hipStream_t, int, FlowWaits);
template int solve_impl<double, KIND_CHOL>(const double*, int64_t, int64_t, double*, int64_t, int64_t, void*, size_t, hipStream_t, int, FlowWaits);
template int solve_impl<float, KIND_CHOL>(const float*, int64_t, int64_t, float*, int64_t, int64_t, void*, size_t, hipStream_t, int, FlowWaits);

}  // namespace dla
