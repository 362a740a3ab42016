// The host-callable parts of flow_kernel.hpp, for tests that need no GPU.
#include "flow_kernel.hpp"

extern "C" {
// The slots that the waits of one workgroup hand over in, in their order.
void flow_host_slots(int waits, int* slot) {
  dla::FlowSlots s;
  for (int i = 0; i < waits; ++i) slot[i] = s.next();
}
}
