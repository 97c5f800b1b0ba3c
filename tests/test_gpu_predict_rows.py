"""de_sur_predict on rows that end with the buffer: the last row holds its D
coordinates and no padding behind them.
"""
import numpy as np
import pytest

from tests import test_gpu_surrogate as sur
from tests.gpu_helpers import HI, LO, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


# last groups of one, two and three coordinates, rows of 16-byte groups; a last
# tile of one row, a full one and one between
@pytest.mark.parametrize("D,H,n", [(33, 32, 129), (62, 128, 128),
                                   (99, 256, 200), (130, 96, 70)])
def test_last_row_without_padding(D, H, n):
    import torch
    from paper_2405_16551_amd import de as lib
    s, _ = sur.make_sur(runs=1, NP=64, D=D, hidden=H, steps=3, warmup_gens=1)
    s.generation(3)
    ld = (D + 3) // 4 * 4
    X = np.random.default_rng(n).uniform(LO, HI, (n, D)).astype(np.float32)
    buf = torch.empty((n - 1) * ld + D, dtype=torch.float32, device=s.device)
    torch.as_strided(buf, (n, D), (ld, 1)).copy_(torch.from_numpy(X))
    y = torch.empty(n, dtype=torch.float32, device=s.device)
    lib._check(lib._lib.de_sur_predict(s.handle, 0, buf.data_ptr(), n, ld,
                                       y.data_ptr(), s._s()), "de_sur_predict")
    np.testing.assert_array_equal(host(y), host(s.predict(0, X)))
    s.close()


# tiles of 64 rows while there are fewer than three per compute unit, then of
# 128: rows at both sides of the line (768 tiles of 64) equal a few of them
@pytest.mark.parametrize("D,H", [(30, 32), (64, 64), (90, 128), (100, 256)])
def test_tile_heights_agree(D, H):
    s, _ = sur.make_sur(runs=1, NP=64, D=D, hidden=H, steps=3, warmup_gens=1)
    s.generation(3)
    X = np.random.default_rng(D).uniform(LO, HI, (49153, D)).astype(np.float32)
    high = host(s.predict(0, X))
    low = host(s.predict(0, X[:767 * 64]))
    np.testing.assert_array_equal(low, high[:len(low)])
    np.testing.assert_array_equal(host(s.predict(0, X[-65:])), high[-65:])
    s.close()
