// The library's rules that are plain functions of sizes, for a process without a GPU (tests/test_rules.py).
#include "../../paper_2005_14469_amd/csrc/gcoo_band.hpp"
#include "../../paper_2005_14469_amd/csrc/gcoo_spdm_launch.hpp"

extern "C" {

int32_t band_tests(int32_t lists) { return gcoo::band_tests(lists); }
int64_t band_test_from(int64_t w, int32_t lists) { return gcoo::band_test_from(w, lists); }
int32_t band_test_says(int64_t w, int32_t lists) { return gcoo::band_test_says(w, lists); }

int32_t rows_turn(int32_t wg, int64_t row_wgs, int64_t tiles) { return gcoo::rows_turn(gcoo::rows_turns(row_wgs, tiles), wg); }

}  // extern "C"
