// Host side of gemm_wide_kernel: which tile a launch takes, and the launch.
#include "dla_codes.hpp"
#include "gemm_dispatch.hpp"
#include "gemm_wide_kernel.hpp"

namespace dla {

// The tiles: X(waves along m, along n, 16 x 16 blocks per wave along m, along n, rate).  rate: TFLOP/s of a
// 4096 x 4096 x 1024 product in fp64 (fp32 ranks them the same way, 93, 107, 110, 115).
#define DLA_WIDE_MENU(X) \
  X(2, 2, 1, 1, 57)      \
  X(2, 2, 2, 1, 65)      \
  X(4, 2, 1, 2, 72)      \
  X(4, 2, 2, 2, 73)

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

// The kernel's element offsets inside a tile are 32-bit, and what it loads of a row with its columns in memory is whole
// runs of 16 bytes: rows shorter than one are gemm_kernel's.
template <typename T>
bool gemm_wide_fits(int op, const GemmGroup<T>& g) {
  constexpr int PER = WideVec<T>::PER;
  if (op != OP_ASSIGN && op != OP_SUB && op != OP_SUB_TN) return false;
  for (int q = 0; q < g.nprob; ++q) {
    const GemmProblem<T>& p = g.prob[q];
    if (p.lda > (1 << 24) || p.ldb > (1 << 24) || p.N < PER || (op == OP_SUB_TN && p.M < PER)) return false;
  }
  return true;
}

// A launch lasts as long as its busiest compute unit: rounds = tiles / 256 rounded up, each one tile at the tile's own
// rate; the least wins.  (fp64 G of the extralarge 3mm, 1600 x 2200: 64 x 32 tiles, 6.7 per unit, 208 us; 64 x 64, 3.4
// per unit, 214 us; 128 x 64, 1.8 per unit, 213 us.  E|F: 64 x 64, 6.8 per unit, 487 us; 64 x 32 530; 128 x 64 545.)
template <typename T>
int launch_gemm_wide(int op, GemmGroup<T>& g, hipStream_t st) {
  double best = 0.0;
  int pick = -1, at = 0;
#define DLA_CASE(WM, WN, FM, FN, RATE)                                                       \
  {                                                                                          \
    constexpr int TM = WM * FM * 16, TN = WN * FN * 16;                                      \
    int64_t tiles = 0;                                                                       \
    for (int q = 0; q < g.nprob; ++q)                                                        \
      tiles += (int64_t)((g.prob[q].M + TM - 1) / TM) * ((g.prob[q].N + TN - 1) / TN);       \
    const double cost = (double)((tiles + 255) / 256) * (TM * TN) / RATE;                    \
    if (pick < 0 || cost < best) {                                                           \
      best = cost;                                                                           \
      pick = at;                                                                             \
    }                                                                                        \
    ++at;                                                                                    \
  }
  DLA_WIDE_MENU(DLA_CASE)
#undef DLA_CASE
  at = 0;
#define DLA_CASE(WM, WN, FM, FN, RATE) \
  if (at++ == pick) return launch_wide_tile<T, WM, WN, FM, FN>(op, g, st);
  DLA_WIDE_MENU(DLA_CASE)
#undef DLA_CASE
  return DLA_ERR_UNSUPPORTED_PARAMS;
}

template bool gemm_wide_fits<double>(int, const GemmGroup<double>&);
template bool gemm_wide_fits<float>(int, const GemmGroup<float>&);
template int launch_gemm_wide<double>(int, GemmGroup<double>&, hipStream_t);
template int launch_gemm_wide<float>(int, GemmGroup<float>&, hipStream_t);

}  // namespace dla
