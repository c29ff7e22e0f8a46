"""Detection on grids of the caller's, at the edges of its passes over the lags.

The argmax kernel runs 1024 threads with 16 column maxima each in registers:
above 16384 lags it reads them again for the second peak.  The block sums of the
mean come from blocks of 256 lags.  Grids around those sizes, and the smallest,
with ties, with maxima in the first and the last lag, and with values that are
not numbers, against the float64 oracle.
"""
import math

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")


def _detect(c, grid, prns, spc):
    n_prn, nd, N = grid.shape
    d_g = torch.from_numpy(grid).cuda()
    d_p = torch.zeros(n_prn * 48, dtype=torch.uint8, device="cuda")
    c.peaks(d_g.data_ptr(), prns, nd, N, spc, -300.0, 100.0, d_p.data_ptr(), torch.cuda.current_stream())
    torch.cuda.synchronize()
    return d_p.cpu().numpy().view(G.PEAK_DTYPE)


@pytest.mark.parametrize("N", [3, 63, 64, 65, 1023, 1024, 1025, 16383, 16384, 16385, 33000, 300001])
@pytest.mark.parametrize("nd", [1, 9])
def test_records_against_oracle(N, nd):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(N + nd)
    g = rng.uniform(0.5, 1.0, (5, nd, N)).astype(np.float32)
    g[0, nd - 1, N - 1] = 9.0                      # last lag, last row
    g[1, nd // 2, 0] = g[1, nd // 2, N - 1] = 8.0  # tie over lag: the first
    g[2, nd // 2, N // 2] = 7.0
    g[2, 0, N - 1] = 6.5                           # second peak in the last lag
    g[3, :, :] = 1.0                               # flat: a tie of all lags
    prns = [4, 8, 15, 16, 23]
    spc = 0 if N < 8 else 3
    with G.Context(0) as c:
        got = _detect(c, g, prns, spc)
    for i in range(5):
        r, o = O.peak_one(g[i].astype(np.float64), prns[i], spc, 2.5, -300.0, 100.0), got[i]
        assert (o["prn"], o["doppler_bin"], o["code_phase"], bool(o["detected"])) == \
            (r.prn, r.doppler_bin, r.code_phase, r.detected), i
        assert o["peak"] == np.float32(r.peak) and o["second"] == np.float32(r.second)
        assert o["ratio"] == np.float32(o["peak"]) / np.float32(o["second"])
        # column sums in row order, trees over 256 lags, threads' sums over every
        # 1024th block, a tree over 1024 threads, the division
        depth = nd + 8 + -(-N // (256 * 1024)) + 10 + 2
        assert abs(o["mean"] - r.mean) <= depth * 2.0 ** -24 * r.mean
        assert abs(o["doppler_hz"] - r.doppler_hz) < 1e-9
        assert abs(o["code_phase_frac"] - r.code_phase_frac) < 1e-9 * max(1, N / 1024)


@pytest.mark.parametrize("N", [40, 20000])
def test_values_that_are_no_numbers(N):
    """No ordered maximum leaves bin and phase 0; a NaN or an infinity elsewhere
    does not move a maximum that is ordered."""
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    g = np.ones((4, 3, N), np.float32)
    g[0, :, :] = np.nan
    g[1, 1:, 5] = np.nan
    g[1, 2, N - 3] = 4.0
    g[2, :, :] = -np.inf
    g[3, 1, N - 1] = np.inf
    with G.Context(0) as c:
        got = _detect(c, g, [1, 2, 3, 4], 2)
    assert [(int(o["doppler_bin"]), int(o["code_phase"])) for o in got] == [(0, 0), (2, N - 3), (0, 0), (1, N - 1)]
    assert got[0]["peak"] == -np.inf and got[0]["second"] == 0.0 and math.isnan(got[0]["mean"])
    assert got[1]["peak"] == 4.0 and got[1]["second"] == 1.0 and got[1]["ratio"] == 4.0
    assert got[2]["peak"] == -np.inf and got[2]["second"] == 0.0
    assert got[3]["peak"] == np.inf and got[3]["second"] == 1.0 and got[3]["detected"]
    assert math.isnan(got[0]["code_phase_frac"]) and math.isnan(got[2]["code_phase_frac"])
