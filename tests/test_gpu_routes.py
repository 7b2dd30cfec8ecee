"""Operations whose passes depend on more than the grid: on 3600^2 a PSF or a
field of many rows takes the five digit passes (in wavelength groups), one of
few rows the three of the small grids.  Both against the FP64 oracle (fields
1e-5, intensities 2e-5), the groups bitwise against one wavelength at a time,
and the launch counts of the timed passes show which ran."""

import os

import numpy as np
import pytest

import oracle
from oracle import asm
from paper_2505_22313_amd import workloads as wl
from _close import FIELD_ELEM, INTENSITY_ELEM, assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

asm.WORKERS = min(16, os.cpu_count() or 1)


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_22313_amd import api as _api
    yield _api
    _api.default_context(0).release_workspaces()
    torch.cuda.empty_cache()


def launches(api, fn):
    ctx = api.default_context(0)
    ctx.profile_enable(True)
    try:
        fn()
        return {k: v[0] for k, v in ctx.profile_read().items()}
    finally:
        ctx.profile_enable(False)


@pytest.mark.parametrize("ny,nx,k,mode,five", [
    (2701, 2699, 2, "crop", True), (3600, 3599, 5, "crop", True), (1500, 1801, 3, "full", True),
    (2000, 1801, 2, "crop", False), (1801, 3600, 1, "crop", False), (900, 33, 1, "full", False),
])
def test_psf_3600(api, ny, nx, k, mode, five):
    rng = np.random.default_rng(ny + nx + k)
    lams = np.linspace(0.42, 0.68, k) if k > 1 else np.array([0.55])
    w = np.linspace(0.5, 1.5, k).astype(np.float32)
    nidx = wl.cauchy_index(lams)
    prob = api.Problem((ny, nx), 3600, 0.5, 700.0, lams, nidx, weights=w, out_mode=mode)
    hn = rng.uniform(0.0, 1.2, (ny, nx)).astype(np.float32)
    an = rng.uniform(0.3, 1.0, (ny, nx)).astype(np.float32)
    h, a = torch.from_numpy(hn).cuda(), torch.from_numpy(an).cuda()
    got = api.psf(h, prob, amp=a)
    assert torch.equal(got, api.psf(h, prob, amp=a, group=1))
    count = launches(api, lambda: api.psf(h, prob, amp=a))
    assert (count["pass_b_fwd"] > 0) == five and count["pass_c"] == k
    assert count["pass_a_fwd"] == (-(-k // 4) if five else k)
    want = oracle.psf(hn, 0.5, 700.0, 3600, lams, nidx, weights=w, amp=an, out_mode=mode)
    assert_close(got, want, 2e-5, INTENSITY_ELEM, "psf")


@pytest.mark.parametrize("ny,nx,mode,five", [(2701, 2699, "crop", True), (1801, 77, "full", True),
                                             (2700, 1801, "crop", False)])
def test_field_3600(api, ny, nx, mode, five):
    rng = np.random.default_rng(ny + nx)
    u = (rng.standard_normal((ny, nx)) + 1j * rng.standard_normal((ny, nx))).astype(np.complex64)
    prob = api.Problem((ny, nx), 3600, 0.5, -900.0, [0.55], [1.46], out_mode=mode)
    ud = torch.from_numpy(u).cuda()
    got = api.propagate(ud, prob)
    count = launches(api, lambda: api.propagate(ud, prob))
    assert (count["pass_b_fwd"] > 0) == five
    want = oracle.propagate(u, 3600, 0.5, 0.55, -900.0, out_mode=mode)
    assert_close(got, want, 1e-5, FIELD_ELEM, "field")
