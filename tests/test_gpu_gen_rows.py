"""General-rate searches around the rule that sends 4096-point transforms to rows.

Above 256 (PRN, bin) items a search at N = 1366..2047 (one segment) or 2049..2730 (two)
runs in rows, two PRNs to a workgroup; up to 256 it runs in one piece.  Item counts just at
and just above the line, odd PRN counts and a single PRN (a workgroup's second transform
then repeats the last PRN and must not be written: floats behind the grid are checked), in
the three formats, with code-Doppler shifts.  Against the oracle's direct correlation within
the FP32 grid tolerance of the other general-rate tests.
"""
import numpy as np
import pytest

import oracle as O
import synth
from parity import assert_grid_close, compare_detections, compare_refinement, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

CASES = [
    # N, format, T_coh, blocks, PRNs, bins, code Doppler
    (2730, O.CPLX_I8, 1, 2, 31, 9, 1),
    (2500, O.REAL_2BIT_PACKED, 2, 1, 31, 9, 0),
    (2049, O.REAL_I8, 1, 1, 1, 257, 0),
    (2049, O.CPLX_I8, 1, 2, 32, 8, 0),          # 256 items: in one piece
    (2051, O.CPLX_I8, 1, 1, 29, 9, 1),
    (1366, O.REAL_I8, 1, 2, 31, 9, 1),
    (2000, O.REAL_2BIT_PACKED, 1, 1, 37, 7, 0),
]


@pytest.mark.parametrize("case", CASES, ids=["%d_fmt%d_P%d_K%d_cd%d" % (c[0], c[1], c[4], c[5], c[6]) for c in CASES])
def test_rows_of_4096_match_direct_oracle(case):
    N, fmt, Tc, Nnc, n_prn, nd, cd = case
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs = N * 1000
    f_if = 0.0 if fmt == O.CPLX_I8 else fs / 4.0
    step = 250.0
    lo = 60000.0 if cd else -step * (nd // 2)  # at 60 kHz a block drifts by up to a tenth of a sample per ms
    hi = lo + step * (nd - 1)
    prns = list(range(38 - n_prn, 38)) if n_prn > 1 else [37]
    assert O.n_doppler(lo, hi, step) == nd
    pl = [synth.Planted(prn=prns[-1], code_phase=N - 3, doppler_hz=lo + step * (nd // 2), cn0_dbhz=52.0,
                        carrier_phase=1.0)]
    snap = synth.make_snapshot(N + nd, fmt, fs, f_if, Tc * Nnc + 0.2, pl, O.ca_code)
    d_x = torch.from_numpy(np.ascontiguousarray(snap.samples)).cuda()
    cells = n_prn * nd * N
    d_grid = torch.full((cells + nd * N + 16,), -7.0, dtype=torch.float32, device="cuda")
    d_pk = torch.zeros(n_prn * 48, dtype=torch.uint8, device="cuda")
    req = G.make_request(d_x.data_ptr(), fmt, snap.n, fs, f_if, prns, lo, hi, step, Tc, Nnc, d_grid.data_ptr(),
                         d_pk.data_ptr())
    with G.Context(0) as c:
        c.set("code_doppler", cd)
        c.acquire_device(req, torch.cuda.current_stream())
        torch.cuda.synchronize()
    out = d_grid.cpu().numpy()
    assert np.all(out[cells:] == -7.0)
    grid = out[:cells].reshape(n_prn, nd, N)
    pk = d_pk.cpu().numpy().view(G.PEAK_DTYPE)
    P = O.grid_direct(snap.samples, fmt, fs, f_if, prns, lo, step, nd, Tc, Nnc, code_doppler=bool(cd))
    worst = assert_grid_close(grid, P)
    ref = O.peaks(P, prns, O.chip_exclusion(fs), 2.5, lo, step)
    compare_detections(pk, ref, P)
    compare_refinement(pk, ref, P, grid, lo, step)
    log("rows N=%d, %d x %d: max mixed error %.3e" % (N, n_prn, nd, worst))
