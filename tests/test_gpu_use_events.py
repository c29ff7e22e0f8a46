"""Calls of one context that alternate between the two ways their metadata reaches the device
(a kernel's argument, a copy) while its buffers grow, without a wait between them: a buffer is
freed only after the last call that used it, whichever event marked that one.  Every grid
equals, bit for bit, the same call's in a context of its own."""
import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

FS, N = 1023000, 1023


def test_alternating_routes_with_growing_buffers():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    snap = synth.make_snapshot(5, O.CPLX_I8, FS, 0.0, 4.5, [], O.ca_code)
    d_x = torch.from_numpy(np.ascontiguousarray(snap.samples)).cuda()
    s = torch.cuda.current_stream()

    def call(c, bins, prns):
        grid = torch.full((len(prns), bins, N), -1.0, device="cuda")
        pk = torch.zeros(len(prns) * 48, dtype=torch.uint8, device="cuda")
        c.acquire_device(G.make_request(d_x.data_ptr(), O.CPLX_I8, snap.n, FS, 0.0, prns, -bins / 2.0, bins / 2.0 - 1.0,
                                        1.0, 1, 4, grid.data_ptr(), pk.data_ptr()), s)
        return grid, pk

    calls = [(4, [3]), (700, [3, 8]), (60, [1, 2, 9, 30]), (1400, [5]), (8, [31] * 12), (2600, [7, 7]), (100, [4]), (4000, [6])]
    with G.Context(0) as c:
        got = [call(c, b, p) for b, p in calls]
        torch.cuda.synchronize()
    for (b, p), (grid, pk) in zip(calls, got):
        with G.Context(0) as c:
            want, want_pk = call(c, b, p)
            torch.cuda.synchronize()
        assert torch.equal(grid, want) and torch.equal(pk, want_pk), b
