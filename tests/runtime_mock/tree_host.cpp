// The host-callable arithmetic of simgraph_tree.hip.
#include "simgraph_tree.hip"

namespace stag {
stag_status radix_sort_pairs_u32(const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, int64_t, int, Workspace&,
                                 hipStream_t) {
  return STAG_OK;
}
}  // namespace stag

extern "C" int32_t stag_simgraph_draws_per_node(int64_t, int32_t) { return 1; }
extern "C" uint32_t tree_row_of_draw(uint32_t e, uint32_t s) { return stag::quotient(e, stag::div_by(s)); }
