"""Rules by which a sort takes one form or another, from the sources themselves and from what a call enqueues (no GPU)."""
import ctypes
import os
import subprocess

import pytest

from test_launches_cpu import VALS, VALS_TMP, run, sort    # noqa: F401  (run: a fixture)

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("sort_rules") / "libshim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-Wextra", "-Werror", "-o", so, os.path.join(HERE, "sort_rules_shim.cpp")], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("bits", [1, 10, 11, 12, 14, 16, 20, 31, 32])
def test_more_keys_than_values_are_not_sorted_by_bins(rules, bits):
    """Bins of more than one key on average lose to the two passes that so few bits take."""
    for n in (1, 2, 2049, 2500, 4096, 4097, 7812, 13_671, 16_384, 20_480):
        assert rules.shim_bins_suffice(n, bits) == (n <= 1 << bits), (n, bits)


@pytest.mark.parametrize("n,large", [(256 * 18_000 + 255, False), (256 * 18_001, True), (256 * 20_480 + 255, True), (256 * 20_481, False)])
def test_which_pairs_have_the_kernel_with_20_rows(run, n, large):    # noqa: F811
    """Buckets of 18,433 to 20,480 pairs, on more bits than two passes sort."""
    widths = (17, 24, 25, 32)
    v = dict(vals=VALS, vals_tmp=VALS_TMP)
    got = run([sort(n, bits, **v) for bits in widths] + [sort(n, bits) for bits in widths])
    names = [[k.kernel.split("<")[0] for k in launched if k.kernel.startswith("block_sort")] for rc, launched in got]
    assert names[:4] == [["block_sort_pairs20_kernel" if large and bits > 24 else "block_sort_kernel"] for bits in widths]
    assert names[4:] == [["block_sort_kernel"]] * 4
