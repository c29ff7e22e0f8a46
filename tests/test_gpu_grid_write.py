"""The correlation kernels' grid write at any address a float may have.

Runs of four consecutive phases are written 16 bytes at a time.  Rates with 1 to
16 samples per chip (runs that are and are not multiples of four, items that end
inside a bin), in the three precisions: a grid that starts 1 to 3 floats past a
16-byte address holds the values of one that does not, and the floats around it
stay.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1309_0052_amd")

PRNS, BINS, BLOCKS = [5, 9, 30], 3, 3


@pytest.mark.parametrize("precision", ["FP32", "FP16", "FP16_PFA"])
@pytest.mark.parametrize("spc", [1, 2, 3, 4, 5, 7, 8, 12, 16])
def test_unaligned_grid(precision, spc):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fs, N = 1023000 * spc, 1023 * spc
    rng = np.random.default_rng(spc)
    x = torch.from_numpy(rng.integers(-40, 41, size=2 * BLOCKS * N, dtype=np.int8)).cuda()
    cells = len(PRNS) * BINS * N
    got = []
    with G.Context(0, precision=getattr(G, "GNSS_" + precision)) as c:
        for off in range(4):
            buf = torch.full((cells + 8,), -7.0, device="cuda")
            assert buf.data_ptr() % 16 == 0
            pk = torch.zeros(len(PRNS) * 48, dtype=torch.uint8, device="cuda")
            c.acquire_device(G.make_request(x.data_ptr(), O.CPLX_I8, BLOCKS * N, fs, 0.0, PRNS, -500.0, 500.0, 500.0, 1,
                                            BLOCKS, buf.data_ptr() + 4 * off, pk.data_ptr()),
                             torch.cuda.current_stream())
            torch.cuda.synchronize()
            b = buf.cpu().numpy()
            assert np.all(b[:off] == -7.0) and np.all(b[off + cells:] == -7.0)
            got.append(b[off:off + cells])
    assert np.all(got[0] >= 0.0) and got[0].any()
    for g in got[1:]:
        assert np.array_equal(g, got[0])
