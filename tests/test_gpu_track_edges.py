"""Tracking correlators at the edges of their loops, bit for bit.

Epochs around one workgroup stride (256 samples) and around the part of an epoch
that int32 sums hold (1023 strides and a remainder), channel counts around the
groups of four, the largest code rate (256 samples advance exactly one period)
and the smallest and largest early-late offsets, full-scale samples of both
signs, in the three formats with starts inside a packed byte.  Exact integers on
both sides.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

CASES = [
    # format, channels, start, epoch length, epochs, spacing, largest code rate
    (O.CPLX_I8, 1, 0, 1, 5, 1.0, False),
    (O.REAL_2BIT_PACKED, 4, 3, 255, 7, 1e-9, False),
    (O.REAL_I8, 5, 1, 256, 6, 1.0, True),
    (O.CPLX_I8, 8, 2, 257, 5, 0.5, True),
    (O.REAL_2BIT_PACKED, 9, 6, 1023 * 256, 2, 0.5, False),
    (O.CPLX_I8, 3, 1, 1023 * 256 + 255, 1, 0.25, True),
    (O.CPLX_I8, 2, 5, 1024 * 256 + 1, 2, 1.0, False),
]


@pytest.mark.parametrize("case", CASES, ids=["fmt%d_ch%d_len%d" % (c[0], c[1], c[3]) for c in CASES])
def test_track_edges_match_oracle(case):
    fmt, n_ch, start, elen, n_ep, spacing, fastest = case
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(elen + n_ch)
    fs, n = 4092000, start + elen * n_ep
    if fmt == O.CPLX_I8:
        x = rng.choice(np.array([-128, -127, -1, 0, 127], np.int8), 2 * n)
    elif fmt == O.REAL_I8:
        x = rng.choice(np.array([-128, 127], np.int8), n)
    else:
        x = rng.integers(0, 256, (n + 3) // 4).astype(np.uint8)
    rate = 1023.0 * fs / 256.0 if fastest else 1023000.0
    chans = [O.Channel(prn=1 + 5 * i % 37, carrier_hz=float(rng.uniform(-2e6, 2e6)), carrier_phase=float(rng.uniform(0, 1)),
                       code_phase=float(rng.uniform(0, 1023)), code_rate=rate, spacing=spacing) for i in range(n_ch)]
    ref = O.track(x, fmt, fs, chans, start, elen, n_ep)
    d_x = torch.from_numpy(x).cuda()
    d_o = torch.full((n_ch * n_ep * 6,), -7, dtype=torch.int64, device="cuda")
    req = G.make_track_request(d_x.data_ptr(), fmt, n, fs, chans, start, elen, n_ep, d_o.data_ptr())
    with G.Context(0) as c:
        c.track_device(req, torch.cuda.current_stream())
        torch.cuda.synchronize()
    assert np.array_equal(d_o.cpu().numpy().reshape(n_ch, n_ep, 3, 2), ref)
