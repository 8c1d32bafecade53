"""Which large sorts take two passes and small buckets: kernels and grids (no GPU: see launch_recorder.py; where their scratch lies: test_sort_rules_cpu.py)."""
import pytest

from test_launches_cpu import VALS, VALS_TMP, run, sort    # noqa: F401  (run: a fixture)

FEW, MOST = 3 << 23, 4700 << 14


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("policy", [0, 1])                # 1: tiles by ticket
def test_launches_of_large_sorts(run, pairs, policy):    # noqa: F811
    v = dict(vals=VALS, vals_tmp=VALS_TMP) if pairs else {}
    sizes = [(n, bits) for n in (FEW - 1, FEW, (4701 << 13) - 1, 4701 << 13, MOST, MOST + 1, 1 << 30) for bits in (16, 24, 25, 26, 32)]
    got = run([("tcuscan_set_chain_policy", [policy])] + [sort(n, bits, **v) for n, bits in sizes])[1:]
    for (n, bits), (rc, launched) in zip(sizes, got):
        log = 13 if n >> 13 <= 4700 else 14
        names = [k.kernel.split("<")[0] for k in launched if "fill_zero" not in k.kernel]
        if not (FEW <= n <= MOST and bits >= 25 and bits >= log + 12):
            assert rc == 0 and names == ["digit_histograms_kernel"] + ["digit_pass_kernel"] * -(-bits // 8), (n, bits)
            continue
        tiles, ranges = -(-n // 16384), 1 << (log - ((log + 2) // 2 if pairs else log // 2))
        want = [("fine_sample_kernel", 65), ("fine_count_kernel", 512), ("fine_judge_kernel", ranges), ("fine_start_kernel", 256),
                ("digit_pass_kernel", tiles), ("digit_pass_kernel", tiles + ranges), ("digit_pass_kernel", tiles), ("digit_pass_kernel", tiles),
                ("fine_sort_kernel", 1 << log), ("fine_sort_large_kernel", 512)]
        assert rc == 0 and [(k.kernel.split("<")[0], k.grid) for k in launched] == want, (n, bits)
