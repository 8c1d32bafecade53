"""Compaction of large calls, whose masks are counted a generation of tiles ahead: sizes at the edge of the rule and of tiles,
masks that are all ones, all zeros or change from tile to tile, misaligned arrays, tickets and capture."""
import numpy as np
import pytest

from paper_2411_17887_amd import tcuscan

pytestmark = pytest.mark.gpu

FROM, TILE = 1 << 25, 16384


def make(n, mask, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    i = torch.arange(n, device="cuda")
    m = {"half": lambda: torch.rand(n, generator=g, device="cuda") < 0.5, "ones": lambda: i >= 0, "none": lambda: i < 0,
         "one_in_all": lambda: i == n - 1, "tiles": lambda: (i // TILE) % 3 != 1, "first": lambda: i < 600 * TILE + 7}[mask]()
    return v, m.to(torch.int8)


def check(v, m, out, count, n):
    import torch
    want = v[m != 0]
    assert int(count) == want.numel()
    assert torch.equal(out[: want.numel()], want) and bool((out[want.numel():n] == -5).all())


@pytest.mark.parametrize("mask", ["half", "ones", "none", "one_in_all", "tiles", "first"])
@pytest.mark.parametrize("n", [FROM - 1, FROM, FROM + 1, FROM + TILE - 1, FROM + 3 * TILE])
def test_sizes_and_masks(n, mask):
    import torch
    v, m = make(n, mask, n)
    out, count = torch.full((n,), -5, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    for policy in (0, 1):
        tcuscan.set_chain_policy(policy)
        try:
            out.fill_(-5)
            tcuscan.compact_u32(v, m, out, None, count=count, ws=ws)
            torch.cuda.synchronize()
        finally:
            tcuscan.set_chain_policy(0)
        assert tcuscan.workspace_fault(ws) == 0
        check(v, m, out, count, n)


@pytest.mark.parametrize("off_values,off_mask,off_out", [(1, 0, 0), (0, 1, 0), (0, 16, 3), (3, 5, 1)])
def test_misaligned(off_values, off_mask, off_out):
    import torch
    n = FROM + 12345
    v, m = make(n + 16, "half", 3)
    v, m = v[off_values:off_values + n], m[off_mask % 16:][:n]
    out, count = torch.full((n + 8,), -5, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    tcuscan.compact_u32(v, m, out[off_out:], None, count=count, ws=tcuscan.new_workspace(1, n, "i8"))
    torch.cuda.synchronize()
    check(v, m, out[off_out:], count, n)
    assert bool((out[:off_out] == -5).all())


@pytest.mark.parametrize("off_mask", [16, 48, 4096 + 16])
def test_a_mask_that_starts_inside_its_buffer(off_mask):
    import torch
    n = FROM + 12345
    v, m = make(n + off_mask, "half", 4)
    v, m = v[off_mask:], m[off_mask:]
    out, count = torch.full((n + 3,), -5, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    tcuscan.compact_u32(v, m, out[3:], None, count=count, ws=tcuscan.new_workspace(1, n, "i8"))
    torch.cuda.synchronize()
    check(v, m, out[3:], count, n)
    assert bool((out[:3] == -5).all())


def test_recorded_into_a_graph():
    import torch
    n = FROM + 777
    v, m = make(n, "half", 5)
    out, count = torch.full((n,), -5, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tcuscan.compact_u32(v, m, out, None, count=count, ws=ws)
    for mask in ("tiles", "half", "ones"):
        m.copy_(make(n, mask, 6)[1])
        out.fill_(-5)
        graph.replay()
        torch.cuda.synchronize()
        check(v, m, out, count, n)
        out.fill_(-5)
        tcuscan.compact_u32(v, m, out, None, count=count, ws=ws)          # an eager call on the same workspace between the replays
        torch.cuda.synchronize()
        check(v, m, out, count, n)
