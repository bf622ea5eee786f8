// Test harness (host code): what a mesh handle holds that the C interface does
// not hand out (paper_1908_06909_amd/csrc/common.h).  Built by the tests with
// hipcc; the library itself never uses this file.
#include "common.h"

// The longest edge that the walk's sign bound is taken from.
extern "C" float probe_edge_max(const void* mesh) { return static_cast<const tct_mesh*>(mesh)->edge_max; }
