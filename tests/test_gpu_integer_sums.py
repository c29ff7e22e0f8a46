"""FP32 sums over blocks whose powers are whole numbers.

Samples of few bits, a real IF at a quarter of the rate and the bin at 0 Hz: every carrier
value is +-4096 or 0, so a block's correlation and its power are integers (times the table's
scale).  As long as the transforms keep the powers whole multiples of a power of two, sums
below 2^24 stay on that grid and round away the transforms' own error instead of adding it
up; otherwise equal blocks (a satellite's) round the same way at every addition, and
256 of them are up to 256 half units of 2^-24 off.  The bound is the transforms' error of one
block, four times sqrt(11) roundings of 0.6 2^-24 in amplitude, twice that in power: 1e-6.
"""
import numpy as np
import pytest

import oracle as O
import synth
from parity import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")


@pytest.mark.parametrize("fs,fmt", [(1023000, O.REAL_I8), (2046000, O.REAL_2BIT_PACKED), (4092000, O.REAL_I8),
                                    (2000000, O.REAL_I8), (2500000, O.REAL_I8), (5000000, O.REAL_2BIT_PACKED)])
def test_whole_number_powers_do_not_drift(fs, fmt):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, blocks, prns = fs // 1000, 256, [5, 17, 21, 30]
    pl = [synth.Planted(prn=p, code_phase=(331 * p) % N, doppler_hz=0.0, cn0_dbhz=30.0 + i, carrier_phase=0.7 * i)
          for i, p in enumerate(prns)]
    snap = synth.make_snapshot(fs // 1000, fmt, fs, fs / 4.0, blocks + 0.1, pl, O.ca_code)
    d_x = torch.from_numpy(np.ascontiguousarray(snap.samples)).cuda()
    d_grid = torch.zeros(len(prns) * N, dtype=torch.float32, device="cuda")
    d_pk = torch.zeros(len(prns) * 48, dtype=torch.uint8, device="cuda")
    with G.Context(0) as c:
        c.acquire_device(G.make_request(d_x.data_ptr(), fmt, snap.n, fs, fs / 4.0, prns, 0.0, 0.0, 250.0, 1, blocks,
                                        d_grid.data_ptr(), d_pk.data_ptr()), torch.cuda.current_stream())
        torch.cuda.synchronize()
    grid = d_grid.cpu().numpy().reshape(len(prns), N).astype(np.float64)
    P = O.grid_fft(snap.samples, fmt, fs, fs / 4.0, prns, 0.0, 250.0, 1, 1, blocks)[:, 0]
    assert P.max() < 2.0 ** 24
    peaks = [abs(grid[i].max() - P[i].max()) / P[i].max() for i in range(len(prns))]
    worst = (np.abs(grid - P) / (P + P.mean())).max()
    log("fs %d: peaks off by at most %.2e, cells %.2e" % (fs, max(peaks), worst))
    assert max(peaks) <= 1e-6 and worst <= 1e-6
