"""The upsampling kernels at the edges of their tiles, against the oracle's
one-axis matrices: fine widths around the forward block's 256 columns, coarse
widths around the adjoint block's columns (its 1023 fine columns hold
1023 / s - 5 of them), heights around its 64 rows, odd factors, rows that do
not start on 16-byte boundaries and arrays that do not.  Tolerances as in the
upsampling tests: forward 1e-6, adjoint 1e-5, nearest forward bitwise.
"""

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


def shifted(shape, offset):
    """An uninitialised contiguous float32 tensor `offset` floats past a
    256-byte boundary."""
    n = int(np.prod(shape))
    return torch.full((n + 64,), float("nan"), device="cuda")[offset:offset + n].view(shape)


def kc(s):
    return 1023 // s - 5


SIZES = [(3, 32, 8), (70, 33, 8), (9, kc(8), 8), (65, kc(8) + 1, 8), (2, kc(16), 16),
         (31, kc(16) + 1, 16), (7, kc(7) + 1, 7), (129, 64, 4), (6, kc(2) + 1, 2), (33, 85, 3),
         (5, kc(1) + 1, 1), (64, 63, 5), (1, 300, 8), (300, 1, 12)]


@pytest.mark.parametrize("ncy,ncx,s", SIZES)
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("kind", ["nearest", "lanczos3"])
def test_tile_edges(api, ncy, ncx, s, offset, kind):
    rng = np.random.default_rng(ncy * 1000 + ncx + s)
    wy, wx = ups.axis_matrix(ncy, s, kind), ups.axis_matrix(ncx, s, kind)
    h = rng.uniform(0.0, 1.2, (ncy, ncx)).astype(np.float32)
    fine = shifted((ncy * s, ncx * s), offset)
    got = api.upsample(torch.from_numpy(h).cuda(), s, kind, out=fine).cpu().numpy()
    want = wy @ h.astype(np.float64) @ wx.T
    if kind == "nearest":
        assert np.array_equal(got, want.astype(np.float32))
    else:
        assert_close(got, want, 1e-6, 1e-6, "forward")
    g = shifted((ncy * s, ncx * s), offset)
    g.copy_(torch.from_numpy(rng.standard_normal((ncy * s, ncx * s)).astype(np.float32)))
    got = api.upsample_adjoint(g, s, kind).cpu().numpy()
    assert_close(got, wy.T @ g.cpu().numpy().astype(np.float64) @ wx, 1e-5, 1e-5, "adjoint")
