"""The host side of a call: which kernels it enqueues, for which arguments (no GPU: see launch_recorder.py)."""
import pytest

import launch_recorder

KEYS, TMP, VALS, VALS_TMP, FLAGS, POS, WS = (0x10000 + (i << 36) for i in range(7))
WS_BYTES = 1 << 40


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    shim = launch_recorder.build(tmp_path_factory.mktemp("shim"))
    return lambda calls: launch_recorder.launches(shim, calls)


def sort(n, bits, vals=0, vals_tmp=0, ws=WS):
    return ("tcuscan_split_radix_sort_u32", [KEYS, vals, n, bits, TMP, vals_tmp, FLAGS, POS, ws, WS_BYTES if ws else 0, 0])


@pytest.mark.parametrize("form", [0, 1, 2])
def test_keys_alone_take_the_same_kernels_with_a_scratch_for_payloads(run, form):
    """d_vals_tmp without d_vals is accepted and not used: no kernel that moves payloads is launched."""
    sizes = [(n, bits) for n in (200, 5000, 9000, 16384, 16385, 100_003, 1_000_000, 1 << 22, 6_050_000, 7_000_000, 1 << 30) for bits in (7, 8, 16, 24, 25, 32)]
    got = run([("tcuscan_set_sort_fusion", [form])] + [sort(n, bits, vals_tmp=tmp) for n, bits in sizes for tmp in (0, VALS_TMP)])[1:]
    for at, (n, bits) in enumerate(sizes):
        alone, with_tmp = got[2 * at: 2 * at + 2]
        assert alone[0] == 0 and alone[1], (n, bits)
        assert with_tmp == alone, (n, bits)
