"""Compaction with the positions written by the same kernel: tile edges, pointers at odd places, arrays behind the ends."""
import numpy as np
import pytest

from oracle import apps
from paper_2411_17887_amd import inputs, tcuscan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 8192, 8193, 16383, 16384, 16385, 5 * 16384 + 1021, 300 * 16384 - 7])
@pytest.mark.parametrize("offset", [0, 1])
def test_positions_and_kept_values(n, offset):
    import torch
    for density in (0, 1, None):
        v = inputs.int32_full(n, n + 3).view(np.uint32)
        m = inputs.mask_i8(n, n + 4) if density is None else np.full(n, density, np.int8)
        d_v = torch.from_numpy(np.concatenate([np.zeros(offset, np.int32), v.view(np.int32)])).cuda()[offset:]
        d_m = torch.from_numpy(np.concatenate([np.zeros(offset, np.int8), m])).cuda()[offset:]
        out = torch.full((n + 8,), -5, dtype=torch.int32, device="cuda")
        pos = torch.full((n + offset + 8,), -6, dtype=torch.int32, device="cuda")
        cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        ws = tcuscan.new_workspace(1, n, "i8")
        tcuscan.compact_u32(d_v, d_m, out, pos[offset:], count=cnt, ws=ws)
        torch.cuda.synchronize()
        ref, ref_pos = apps.compact(v, m)
        got = out.cpu().numpy()
        assert int(cnt.item()) == ref.size and np.array_equal(got[:ref.size].view(np.uint32), ref) and np.all(got[ref.size:] == -5)
        p = pos.cpu().numpy()
        assert np.array_equal(p[offset:offset + n], ref_pos) and np.all(p[:offset] == -6) and np.all(p[offset + n:] == -6)
        assert ws is None or tcuscan.workspace_fault(ws) == 0


def test_what_was_refused_is_refused():
    import torch
    n = 20000
    v, out, pos = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3))
    m = torch.zeros(n, dtype=torch.int8, device="cuda")
    L = tcuscan.load()
    stream = torch.cuda.current_stream().cuda_stream
    ws = tcuscan.new_workspace(1, n, "i8")
    need = ws.numel() * 8
    call = lambda p, w, b: L.tcuscan_compact_u32(v.data_ptr(), m.data_ptr(), out.data_ptr(), n, p, 0, w, b, stream)
    assert call(pos.data_ptr(), ws.data_ptr(), need) == tcuscan.OK
    assert call(pos.data_ptr(), ws.data_ptr(), need - 64) == tcuscan.ERR_WORKSPACE
    assert call(pos.data_ptr(), 0, 0) == tcuscan.ERR_WORKSPACE
    assert call(m.data_ptr(), ws.data_ptr(), need) == tcuscan.ERR_INVALID_ARG
    torch.cuda.synchronize()
