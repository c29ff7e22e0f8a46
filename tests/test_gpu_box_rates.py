"""Wipe, fold, boxcar and polyphase split at every number of samples per chip.

One instance of the boxcar per number of samples per chip, in two parts above 8,
with rows of odd stride in LDS and a halo past the last full batch of samples:
each against the definition on the oracle's folded blocks, bit for bit, in the
three formats, with blocks that are read circularly delayed.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

TC, NNC, BINS = 3, 2, 2


@pytest.mark.parametrize("fmt", [O.CPLX_I8, O.REAL_I8, O.REAL_2BIT_PACKED])
@pytest.mark.parametrize("spc", range(1, 17))
def test_every_rate_bit_exact(spc, fmt):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs, N = 1023000 * spc, 1023 * spc
    f_if = 0.0 if fmt == O.CPLX_I8 else fs / 4.0
    lo, step = 300e3, -700e3 if spc % 2 else 45e3  # fast enough to drift by samples within two blocks
    lo, hi, step = min(lo, lo + step), max(lo, lo + step), abs(step)
    n = TC * NNC * N
    rng = np.random.default_rng(10 * spc + fmt)
    if fmt == O.REAL_2BIT_PACKED:
        x = rng.integers(0, 256, size=(n + 3) // 4, dtype=np.uint8)
    else:
        x = rng.integers(-127, 128, size=n * (2 if fmt == O.CPLX_I8 else 1)).astype(np.int8)
    out = torch.full((BINS * NNC * spc * 1024 * 2,), -7, dtype=torch.int32, device="cuda")
    d_x = torch.from_numpy(x).cuda()
    with G.Context(0) as c:
        c.set("code_doppler", 1)
        c.box_fold(G.make_request(d_x.data_ptr(), fmt, n, fs, f_if, [1], lo, hi, step, TC, NNC), out.data_ptr(),
                   torch.cuda.current_stream())
        torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(BINS, NNC, spc, 1024, 2).astype(np.int64)
    folded = O.wipe_fold(x, fmt, fs, f_if, lo, step, BINS, TC, NNC)
    moved = 0
    for k in range(BINS):
        for b in range(NNC):
            shift = O.code_shift(b, TC, N, O.bin_freq(lo, step, k)) % N
            moved += shift != 0
            f = np.roll(folded[k][b], shift, axis=0)
            F = sum(np.roll(f, -t, axis=0) for t in range(spc))
            assert np.array_equal(got[k, b, :, :1023], F.reshape(1023, spc, 2).transpose(1, 0, 2)), (k, b)
            assert not got[k, b, :, 1023].any()
    assert moved
