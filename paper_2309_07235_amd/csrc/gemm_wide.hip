// Host side of gemm_wide_kernel: which tile a launch takes, and the launch.
#include "dla_codes.hpp"
#include "gemm_dispatch.hpp"
#include "gemm_wide_kernel.hpp"

namespace dla {

// The tiles: X(waves along m, along n, 16 x 16 blocks per wave along m, along n, rate in fp64, in fp32, fill).  rate:
// TFLOP/s of whole rounds of tiles, over the three operations at 3000 x 3000 to 6000 x 6000, k = 1024 to 4096.  fill: what
// filling and draining a tile costs, in k, more for the waves with two row blocks, of which fewer fit beside each other.
#define DLA_WIDE_MENU(X)      \
  X(2, 2, 1, 1, 55, 101, 0)   \
  X(2, 2, 2, 1, 64, 117, 16)  \
  X(4, 2, 1, 2, 67, 126, 0)   \
  X(4, 2, 2, 2, 70, 132, 16)

template <typename T, int WM, int WN, int FM, int FN, int OP>
static int launch_wide_op(const GemmGroup<T>& g, hipStream_t st) {
  constexpr int TK = 128 / (int)sizeof(T);
  using S = WideShape<T, WM, WN, FM, FN, TK, OP == OP_SUB_TN>;
  auto kern = gemm_wide_kernel<T, WM, WN, FM, FN, TK, OP>;
  static LdsLimitOnce lds_limit;
  if (!lds_limit.ensure(reinterpret_cast<const void*>(kern), S::BYTES)) return DLA_ERR_HIP;
  hipLaunchKernelGGL(kern, dim3((unsigned)g.total_tiles), dim3(S::NT), S::BYTES, st, g);
  return launch_status(__func__);
}

template <typename T, int WM, int WN, int FM, int FN>
static int launch_wide_tile(int op, GemmGroup<T>& g, hipStream_t st) {
  constexpr int TM = WM * FM * 16, TN = WN * FN * 16;
  int tiles = 0;
  for (int q = 0; q < g.nprob; ++q) {
    GemmProblem<T>& p = g.prob[q];
    p.tiles_m = (p.M + TM - 1) / TM;
    p.tiles_n = (p.N + TN - 1) / TN;
    p.tile_begin = tiles;
    tiles += p.tiles_m * p.tiles_n;
  }
  for (int q = g.nprob; q < kMaxGroup; ++q) g.prob[q] = g.prob[0];
  g.total_tiles = tiles;
  switch (op) {
    case OP_ASSIGN: return launch_wide_op<T, WM, WN, FM, FN, OP_ASSIGN>(g, st);
    case OP_SUB: return launch_wide_op<T, WM, WN, FM, FN, OP_SUB>(g, st);
    case OP_SUB_TN: return launch_wide_op<T, WM, WN, FM, FN, OP_SUB_TN>(g, st);
    default: return DLA_ERR_UNSUPPORTED_PARAMS;
  }
}

// Which products are the wide kernel's.  Its element offsets inside a tile are 32-bit.  And in fp32 a product no deeper
// than a slab, which is traffic of C, is gemm_kernel's (C = A*B, C -= A*B, C -= A^T*B, 4000 x 4000, in us, here against
// there: k = 8 24, 28, 28 against 19, 27, 25; k = 32 20, 26, 26 against 23, 32, 29, but 2047 x 2047 11.3, 11.4, 16.9
// against 11.0, 11.1, 11.2; k = 64 28, 34, 35 against 34, 42, 37).  fp64, k = 8: 25, 41, 42 against 33, 54, 40.
template <typename T>
bool gemm_wide_takes(int op, const GemmGroup<T>& g) {
  if (op != OP_ASSIGN && op != OP_SUB && op != OP_SUB_TN) return false;
  int depth = 0;
  for (int q = 0; q < g.nprob; ++q) {
    const GemmProblem<T>& p = g.prob[q];
    if (p.lda > (1 << 24) || p.ldb > (1 << 24)) return false;
    depth = p.K > depth ? p.K : depth;
  }
  return sizeof(T) == 8 || depth > 32;
}

// A launch lasts as long as its busiest compute unit: rounds = tiles / 256 rounded up, each one tile of the group's mean
// depth, and its fill, at the tile's own rate; the least wins.  Over 140 products of 32 x 400 to 6000 x 6000, k = 8 to 4096,
// all three operations, the choice costs 1.6 % (fp64) and 1.3 % (fp32) more than the best tile in the mean.
template <typename T>
int gemm_wide_pick(const GemmGroup<T>& g, int* tile_m, int* tile_n) {
  double best = 0.0;
  int pick = -1, at = 0;
#define DLA_CASE(WM, WN, FM, FN, RATE64, RATE32, FILL)                                                     \
  {                                                                                                        \
    constexpr int TM = WM * FM * 16, TN = WN * FN * 16;                                                    \
    int64_t tiles = 0;                                                                                     \
    double depth = 0.0;                                                                                    \
    for (int q = 0; q < g.nprob; ++q) {                                                                    \
      const int64_t t = (int64_t)((g.prob[q].M + TM - 1) / TM) * ((g.prob[q].N + TN - 1) / TN);            \
      tiles += t;                                                                                          \
      depth += (double)t * (g.prob[q].K + FILL);                                                           \
    }                                                                                                      \
    const double cost = (double)((tiles + 255) / 256) * (depth / (double)tiles) * (TM * TN) / (sizeof(T) == 8 ? RATE64 : RATE32); \
    if (pick < 0 || cost < best) {                                                                         \
      best = cost;                                                                                         \
      pick = at;                                                                                           \
      *tile_m = TM;                                                                                        \
      *tile_n = TN;                                                                                        \
    }                                                                                                      \
    ++at;                                                                                                  \
  }
  DLA_WIDE_MENU(DLA_CASE)
#undef DLA_CASE
  return pick;
}

template <typename T>
int launch_gemm_wide(int op, GemmGroup<T>& g, hipStream_t st) {
  int tm, tn, at = 0;
  const int pick = gemm_wide_pick(g, &tm, &tn);
#define DLA_CASE(WM, WN, FM, FN, RATE64, RATE32, FILL) \
  if (at++ == pick) return launch_wide_tile<T, WM, WN, FM, FN>(op, g, st);
  DLA_WIDE_MENU(DLA_CASE)
#undef DLA_CASE
  return DLA_ERR_UNSUPPORTED_PARAMS;
}

template bool gemm_wide_takes<double>(int, const GemmGroup<double>&);
template bool gemm_wide_takes<float>(int, const GemmGroup<float>&);
template int gemm_wide_pick<double>(const GemmGroup<double>&, int*, int*);
template int gemm_wide_pick<float>(const GemmGroup<float>&, int*, int*);
template int launch_gemm_wide<double>(int, GemmGroup<double>&, hipStream_t);
template int launch_gemm_wide<float>(int, GemmGroup<float>&, hipStream_t);

}  // namespace dla
