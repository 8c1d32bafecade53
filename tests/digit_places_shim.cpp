// C entry points around paper_2411_17887_amd/csrc/digit_places.h for tests/test_digit_places_cpu.py, which compiles this
// file with g++.
#include "../paper_2411_17887_amd/csrc/digit_places.h"

extern "C" {

unsigned long long shim_place32(unsigned long long before, unsigned start, unsigned i) { return digit_place(digit_base<uint32_t>((uint32_t)before, start), i); }
unsigned long long shim_place64(unsigned long long before, unsigned start, unsigned i) { return digit_place(digit_base<uint64_t>(before, start), i); }
int shim_fits32(unsigned long long before, unsigned count, unsigned n) { return digit_range_fits<uint32_t>((uint32_t)before, count, n) ? 1 : 0; }
int shim_fits64(unsigned long long before, unsigned count, unsigned n) { return digit_range_fits<uint64_t>(before, count, n) ? 1 : 0; }
unsigned shim_bucket_limit(unsigned long long n, unsigned capacity) { return bucket_limit(n, capacity); }

}
