// Test harness (host code): what a mesh handle holds and the walk reads that the
// C interface does not hand out (paper_1908_06909_amd/csrc/common.h).  Built by the tests with
// hipcc; the library itself never uses this file.
#include "common.h"

// The longest edge that the walk's sign bound is taken from.
extern "C" float probe_edge_max(const void* mesh) { return static_cast<const tct_mesh*>(mesh)->edge_max; }

// The walk's read of its local-index remap: loc with the fields of slots 0, 1, 2.
extern "C" unsigned probe_walk_remap(unsigned loc, unsigned k, unsigned back) {
  static constexpr tct::LocRemap table = tct::make_loc_remap();
  return table.v[tct::loc_remap_row(loc, 2 * k) | back];
}
