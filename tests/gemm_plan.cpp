// The choice between the matrix kernels as functions that a test can call.
#include "../paper_2502_20190_amd/csrc/tj_gemm_plan.h"

extern "C" int wide_pair_pays(int tiles, int k) { return tjplan::wide_pair_pays(tiles, k); }
extern "C" int wide_forward_pays(int tiles_i, int tiles_j, int k) { return tjplan::wide_forward_pays(tiles_i, tiles_j, k); }
extern "C" int wide_whole_columns(int tiles_i, int tiles_j) { return tjplan::wide_whole_columns(tiles_i, tiles_j); }
extern "C" int ends_slices(int tiles, int max_batch, int s) { return tjplan::ends_slices(tiles, max_batch, s); }
