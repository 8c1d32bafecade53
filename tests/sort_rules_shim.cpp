// C entry points around the rules of paper_2411_17887_amd/csrc/digit_places.h for tests/test_sort_rules_cpu.py, which compiles this file with g++.
#include "../paper_2411_17887_amd/csrc/digit_places.h"

extern "C" {

int shim_bins_suffice(unsigned n, unsigned bits) { return bins_suffice(n, bits) ? 1 : 0; }

}
