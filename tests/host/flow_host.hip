// The host-callable parts of flow_kernel.hpp, for tests that need no GPU.
#include "flow_kernel.hpp"

extern "C" {
// The slots that the waits of one workgroup hand over in, in their order.
void flow_host_slots(int waits, int* slot) {
  dla::FlowSlots s;
  for (int i = 0; i < waits; ++i) slot[i] = s.next();
}
// The pieces of a launch, five ints each: pass, sum or solution, position, rows, columns; 0 0 -1 0 0: there is no such piece.
int flow_host_pieces(int n, int tiles_n, int* out) {
  const int blocks = (n + dla::kFlowBlock - 1) / dla::kFlowBlock, count = dla::flow_pieces(blocks, tiles_n);
  for (int id = 0; out && id < count; ++id) {
    const dla::FlowPiece f = dla::flow_piece(id, blocks, tiles_n);
    const bool is = dla::flow_piece_is(f, n, blocks);
    const int row[5] = {is && f.back, is && f.sum, is ? f.p : -1, is ? f.rt : 0, is ? f.ct : 0};
    for (int k = 0; k < 5; ++k) out[id * 5 + k] = row[k];
  }
  return count;
}
int flow_host_expected(int n) { return dla::flow_expected(n, (n + dla::kFlowBlock - 1) / dla::kFlowBlock); }
}
