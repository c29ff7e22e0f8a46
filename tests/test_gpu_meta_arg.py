"""Requests whose metadata travels as a kernel argument, and the first that does not.

The request table of a small batch is written by one kernel from its argument;
above 3840 bytes it is copied from pinned staging.  The NCO steps (4 bytes per
Doppler bin) are what grows, so one search over many bins is compared bit for bit
with the same bins searched in parts, on both sides of the limit.  A captured
call replays the table it was captured with, whatever the context ran since.
"""
import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

FS, N = 1023000, 1023


def _request(d_x, n, prns, lo, bins, blocks):
    grid = torch.full((len(prns), bins, N), -1.0, device="cuda")
    pk = torch.zeros(len(prns) * 48, dtype=torch.uint8, device="cuda")
    return G.make_request(d_x.data_ptr(), O.CPLX_I8, n, FS, 0.0, prns, lo, lo + bins - 1.0, 1.0, 1, blocks,
                          grid.data_ptr(), pk.data_ptr()), grid, pk


@pytest.mark.parametrize("bins", [1, 63, 512, 575, 576, 577, 640, 1500])
def test_one_search_equals_its_parts(bins):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    snap = synth.make_snapshot(3, O.CPLX_I8, FS, 0.0, 2.5, [], O.ca_code)
    d_x = torch.from_numpy(snap.samples).cuda()
    s = torch.cuda.current_stream()
    with G.Context(0) as c:
        req, whole, _ = _request(d_x, snap.n, [7, 30], -400.0, bins, 2)
        c.acquire_device(req, s)
        for k in range(0, bins, 100):
            part_req, part, _ = _request(d_x, snap.n, [7, 30], -400.0 + k, min(100, bins - k), 2)
            c.acquire_device(part_req, s)
            torch.cuda.synchronize()
            assert torch.equal(whole[:, k:k + 100], part)


def test_captured_call_replays_its_own_table():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    snaps = [synth.make_snapshot(s, O.CPLX_I8, FS, 0.0, 3.5, [], O.ca_code) for s in (1, 2, 3)]
    d_x = torch.from_numpy(snaps[0].samples.copy()).cuda()
    with G.Context(0) as c:
        req, grid, pk = _request(d_x, snaps[0].n, [4, 9, 20], -20.0, 40, 3)
        other, other_grid, _ = _request(d_x, snaps[0].n, [11], 100.0, 5, 2)
        c.acquire_device(req, torch.cuda.current_stream())  # sizes the workspace
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            c.acquire_device(req, torch.cuda.current_stream())
        for snap in snaps:
            d_x.copy_(torch.from_numpy(snap.samples))
            c.acquire_device(req, torch.cuda.current_stream())
            want, want_pk = grid.clone(), pk.clone()
            c.acquire_device(other, torch.cuda.current_stream())  # another table in the same place
            grid.fill_(-1.0)
            pk.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(grid, want) and torch.equal(pk, want_pk)
