"""The Lanczos-3 kernels where a thread has one column: maps too narrow or too
small for four columns a thread, rows that are not whole 16-byte vectors, at
the edges of the 64-column blocks, of the widest such map, and of blocks of 1
to 16 segments per wavefront; the adjoint at the edges of its 253 and 1021
fine columns.  Against the oracle's one-axis matrices: forward 1e-6, adjoint
1e-5 (rel-L2 and per element), as in the other upsampling tests."""

import numpy as np
import pytest

from oracle import upsample as ups
from _close import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_22313_amd import api as _api
    return _api


def kc(s, cols):
    """Coarse columns of an adjoint block of 256 cols fine columns."""
    return (256 * cols - 3) // s - 5


SIZES = [
    # fine widths around 64 columns and around the widest narrow map, 192
    (300, 63, 1), (301, 64, 1), (29, 65, 1), (500, 21, 3), (7, 22, 3), (2000, 192, 1),
    (2000, 193, 1), (700, 48, 4), (700, 49, 4), (1, 1, 1), (1, 1, 16), (2, 3, 5),
    # 16 segments per wavefront (at s = 5: 12), rows just past a block's
    (1919, 1345, 1), (1920, 1345, 1), (835, 1001, 3), (385, 1001, 5),
    # coarse widths of one adjoint block of one, and of four, columns a thread
    (40, kc(1, 1), 1), (41, kc(1, 1) + 1, 1), (70, kc(8, 1), 8), (69, kc(8, 1) + 1, 8),
    (33, kc(16, 1), 16), (17, kc(16, 1) + 1, 16), (12, kc(7, 1) + 1, 7),
    (6, kc(2, 4), 2), (6, kc(2, 4) + 1, 2), (7, kc(7, 4) + 1, 7), (5, kc(1, 4) + 1, 1),
]


@pytest.mark.parametrize("ncy,ncx,s", SIZES)
def test_one_column_per_thread(api, ncy, ncx, s):
    rng = np.random.default_rng(ncy * 1000 + ncx + s)
    wy, wx = ups.axis_matrix(ncy, s, "lanczos3"), ups.axis_matrix(ncx, s, "lanczos3")
    h = rng.uniform(0.0, 1.2, (ncy, ncx)).astype(np.float32)
    fine = torch.full((ncy * s, ncx * s), float("nan"), device="cuda")
    got = api.upsample(torch.from_numpy(h).cuda(), s, "lanczos3", out=fine)
    assert_close(got, wy @ h.astype(np.float64) @ wx.T, 1e-6, 1e-6, "forward")
    g = rng.standard_normal((ncy * s, ncx * s)).astype(np.float32)
    out = torch.full((ncy, ncx), float("nan"), device="cuda")
    got = api.upsample_adjoint(torch.from_numpy(g).cuda(), s, "lanczos3", out=out)
    assert_close(got, wy.T @ g.astype(np.float64) @ wx, 1e-5, 1e-5, "adjoint")
