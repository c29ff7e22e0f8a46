"""PRN pairs and block batches of the exact-length correlation kernel.

A wave takes two PRNs of a tile at a time, its spectra's 33rd columns in batches
of 16 (block, PRN) pairs: 8 blocks of a pair, 16 of a PRN that is left alone.
Block counts around those batches, with blocks of different exponents and
without any signal, in every tile size and in tiles that the PRNs do not fill:
each PRN's grid against the one it has alone (the same products; the sums over
2 Nnc squares and the matrix products' 32 terms each may be ordered differently,
so each cell within 2 (2 Nnc + 32 * 2) 2^-24 of itself plus, where terms cancel,
of the grid's mean), and against the float64 oracle.
"""
import numpy as np
import pytest

import oracle as O
from parity import grid_error

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

TOLX = 2.0e-2  # the mode's bound against float64 (11 FP16 roundings, see the mode's tests)
PRNS = [3, 17, 31]


def _grid(c, x, fs, blocks, prns, tile):
    c.set("corr_ptile", tile)
    N = fs // 1000
    d_x = torch.from_numpy(x).cuda()
    g = torch.full((len(prns), 3, N), -1.0, device="cuda")
    pk = torch.zeros(len(prns) * 48, dtype=torch.uint8, device="cuda")
    c.acquire_device(G.make_request(d_x.data_ptr(), O.CPLX_I8, x.size // 2, fs, 0.0, prns, -500.0, 500.0, 500.0, 1,
                                    blocks, g.data_ptr(), pk.data_ptr()), torch.cuda.current_stream())
    torch.cuda.synchronize()
    return g.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 15, 16, 17, 33])
@pytest.mark.parametrize("spc", [1, 2, 4, 6])
def test_tiles_equal_single_prns(blocks, spc):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs = 1023000 * spc
    N = fs // 1000
    rng = np.random.default_rng(100 * blocks + spc)
    amp = rng.choice([0, 1, 2, 9, 60, 127], size=blocks)
    x = np.concatenate([rng.integers(-a, a + 1, size=2 * N) for a in amp]).astype(np.int8)
    with G.Context(0, precision=G.GNSS_FP16_PFA) as c:
        alone = np.concatenate([_grid(c, x, fs, blocks, [p], 1) for p in PRNS])
        tiles = {t: _grid(c, x, fs, blocks, PRNS, t) for t in (1, 2, 4, 8)}
    tol = 2 * (2 * blocks + 64) * 2.0 ** -24
    for t, g in tiles.items():
        assert np.all(np.abs(g - alone) <= tol * (alone + alone.mean())), t
    P = O.grid_fft(x, O.CPLX_I8, fs, 0.0, PRNS, -500.0, 500.0, 3, 1, blocks)
    assert np.all(np.isfinite(tiles[2]))
    if amp.any():
        assert grid_error(tiles[2], P) <= TOLX
    else:
        assert not tiles[2].any()
