// The host-callable parts of tile_factor_kernel.hpp, for tests that need no GPU.
#include "factor_kernels.hpp"
#include "tile_factor_kernel.hpp"

extern "C" {
// The tiles of a matrix of nt x nt in the order in which they are taken (kind 0 LU, 1 Cholesky); returns how many.
int tile_host_order(int kind, int nt, int* i, int* j) {
  const int count = kind == 0 ? dla::tile_count<dla::KIND_LU>(nt) : dla::tile_count<dla::KIND_CHOL>(nt);
  for (int id = 0; id < count; ++id) {
    if (kind == 0) dla::tile_of<dla::KIND_LU>(nt, id, i + id, j + id);
    else dla::tile_of<dla::KIND_CHOL>(nt, id, i + id, j + id);
  }
  return count;
}
int tile_host_max() { return dla::kTileMaxNt; }
int tile_host_ring() { return dla::kTileInvRing; }
}
