// The library's rules that are plain functions of sizes, for a process without a GPU (tests/test_rules.py).
#include "../../paper_2005_14469_amd/csrc/gcoo_band.hpp"

extern "C" {

int32_t band_tests(int32_t lists) { return gcoo::band_tests(lists); }
int64_t band_test_from(int64_t w, int32_t lists) { return gcoo::band_test_from(w, lists); }
int32_t band_test_says(int64_t w, int32_t lists) { return gcoo::band_test_says(w, lists); }

}  // extern "C"
