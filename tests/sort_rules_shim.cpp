// C entry points around the rules of paper_2411_17887_amd/csrc/digit_places.h and large_sort_plan.h for tests/large_sort_model.py and
// tests/test_sort_rules_cpu.py, which compile this file with g++.
#include "../paper_2411_17887_amd/csrc/digit_places.h"
#include "../paper_2411_17887_amd/csrc/large_sort_plan.h"

extern "C" {

int shim_bins_suffice(unsigned n, unsigned bits) { return bins_suffice(n, bits) ? 1 : 0; }
int shim_large_wanted(unsigned long long n, int bits) { return large_sort::wanted((size_t)n, bits) ? 1 : 0; }
// log, low, most_tiles, huge_tiles, huge_work, some_most, huge_most, wide_most, work_most, few_most, found, counts, ranges, huge, status, end
void shim_large_plan(unsigned long long n, int vals, unsigned long long *out)
{
    const large_sort::Plan p = large_sort::plan((size_t)n, vals != 0);
    const unsigned long long fields[16] = {(unsigned long long)p.log, (unsigned long long)p.low, p.most_tiles, p.huge_tiles, p.huge_work, p.some_most, p.huge_most, p.wide_most, p.work_most, p.few_most,
                                           p.found, p.counts, p.ranges, p.huge, p.status, p.end};
    for (int i = 0; i < 16; ++i) out[i] = fields[i];
}

}
