"""FP32 searches at chip-rate multiples: every number of samples per chip.

A polyphase vector is transformed as two segments of 512 and 511 values on
1536-point transforms, wiped, folded and split in one kernel whose work item is
a whole (Doppler, block) up to 8 samples per chip and one segment of it above.
Checked at every samples-per-chip value on both sides of that line, in the three
sample formats (packed blocks that start inside a byte among them), with several
coherent milliseconds and with code-Doppler shifts that move samples across the
segment and block boundaries, against the oracle's direct correlation within the
FP32 grid tolerance; and past one group of block sums on an odd rate, where every
PRN tile and workgroup width has to give the same grid.
"""
import numpy as np
import pytest

import oracle as O
import synth
from parity import assert_grid_close, compare_detections, compare_refinement, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")


def _run(c, snap, fs, f_if, prns, lo, hi, step, Tc, Nnc):
    nd, N = O.n_doppler(lo, hi, step), fs // 1000
    d_x = torch.from_numpy(np.ascontiguousarray(snap.samples)).cuda()
    d_grid = torch.zeros(len(prns) * nd * N, dtype=torch.float32, device="cuda")
    d_pk = torch.zeros(len(prns) * 48, dtype=torch.uint8, device="cuda")
    req = G.make_request(d_x.data_ptr(), snap.fmt, snap.n, fs, f_if, prns, lo, hi, step, Tc, Nnc, d_grid.data_ptr(),
                         d_pk.data_ptr())
    c.acquire_device(req, torch.cuda.current_stream())
    torch.cuda.synchronize()
    return d_grid.cpu().numpy().reshape(len(prns), nd, N), d_pk.cpu().numpy().view(G.PEAK_DTYPE).copy()


@pytest.mark.parametrize("spc", range(1, 17))
def test_every_samples_per_chip_matches_direct_oracle(spc):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs, N = spc * 1023000, spc * 1023
    fmt = [O.CPLX_I8, O.REAL_I8, O.REAL_2BIT_PACKED][spc % 3]
    cd = spc % 2
    f_if = 0.0 if fmt == O.CPLX_I8 else fs / 4.0
    Tc, Nnc = 1 + spc % 3, 3
    lo, hi, step = (60000.0, 60500.0, 500.0) if cd else (-500.0, 500.0, 500.0)
    prns = [4, 19, 27][: 1 + spc % 3]
    pl = [synth.Planted(prn=prns[0], code_phase=(511 * spc + 3) % N, doppler_hz=lo + step, cn0_dbhz=52.0)]
    snap = synth.make_snapshot(100 + spc, fmt, fs, f_if, Tc * Nnc + 0.3, pl, O.ca_code)
    with G.Context(0) as c:
        c.set("code_doppler", cd)
        grid, pk = _run(c, snap, fs, f_if, prns, lo, hi, step, Tc, Nnc)
    P = O.grid_direct(snap.samples, fmt, fs, f_if, prns, lo, step, grid.shape[1], Tc, Nnc, code_doppler=bool(cd))
    worst = assert_grid_close(grid, P)
    ref = O.peaks(P, prns, O.chip_exclusion(fs), 2.5, lo, step)
    compare_detections(pk, ref, P)
    compare_refinement(pk, ref, P, grid, lo, step)
    log("spc %d: max mixed error %.3e" % (spc, worst))


def test_launch_shapes_give_the_same_grid_past_one_group():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs, Nnc, prns, lo, hi, step = 3 * 1023000, 258, [2, 3, 9, 14, 30], -250.0, 250.0, 250.0
    snap = synth.make_snapshot(9, O.CPLX_I8, fs, 0.0, Nnc + 0.5, [], O.ca_code)
    grids = []
    with G.Context(0) as c:
        for tile, waves in ((1, 4), (1, 6), (1, 12), (2, 8), (4, 8)):
            c.set("corr_ptile", tile)
            c.set("corr_waves", waves)
            grids.append(_run(c, snap, fs, 0.0, prns, lo, hi, step, 1, Nnc)[0])
    for g in grids[1:]:
        assert np.array_equal(g, grids[0])
    assert_grid_close(grids[0], O.grid_direct(snap.samples, O.CPLX_I8, fs, 0.0, prns, lo, step, grids[0].shape[1], 1, Nnc))
