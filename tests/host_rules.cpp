// C entry points of the host rules (csrc/host_rules.h) for tests/test_host_rules.py.
#include "host_rules.h"

using namespace mgemm;

extern "C" {

int grid_fits_c(int64_t blocks, int64_t threads) { return grid_fits(blocks, threads); }

int list_grid_fits_c(int64_t m, int64_t n) { return list_grid_fits(m, n); }

}  // extern "C"
