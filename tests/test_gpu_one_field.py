"""Grouped wavelengths of the small grids against calls that cannot group: the
library's own entry points with a workspace of exactly one field (timing a call
does not do: it leaves the table grids' groups on).  PSF, saved fields and
gradient are bitwise equal, and where timing leaves groups on its launch counts
show that one call groups and the other does not."""

import numpy as np
import pytest

from paper_2505_22313_amd import _lib as L
from paper_2505_22313_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_22313_amd import api as _api
    return _api


def ptr(t):
    return None if t is None else t.data_ptr()


@pytest.mark.parametrize("m,ny,nx,k,up,amp", [
    (16, 7, 16, 3, 1, False), (64, 33, 20, 5, 1, True), (256, 128, 256, 4, 2, False),
    (1024, 513, 512, 2, 1, True), (2048, 1023, 1025, 6, 1, False),
    (240, 121, 240, 5, 1, True), (720, 359, 361, 4, 1, False), (1440, 700, 720, 3, 4, True),
    ((720, 240), 361, 119, 6, 1, False), ((512, 2048), 255, 1025, 7, 1, True),
    ((5360, 240), 2680, 120, 3, 2, True),
])
def test_group_equals_a_one_field_workspace(api, m, ny, nx, k, up, amp):
    rng = np.random.default_rng(int(np.sum(m)) + k)
    lams = np.linspace(0.42, 0.68, k)
    w = np.linspace(0.5, 1.5, k).astype(np.float32)
    prob = api.Problem((ny, nx), m, 0.5, 400.0, lams, wl.cauchy_index(lams), weights=w, upsample=up)
    h = torch.from_numpy(rng.uniform(0.0, 1.2, prob.h_shape).astype(np.float32)).cuda()
    a = torch.from_numpy(rng.uniform(0.3, 1.0, (ny, nx)).astype(np.float32)).cuda() if amp else None
    g = torch.from_numpy(rng.standard_normal((ny, nx)).astype(np.float32)).cuda()
    ctx = api.default_context(0)
    stream = torch.cuda.current_stream(0).cuda_stream

    def calls(group):
        """psf, psf of the saving call, saved fields, gradient."""
        psf, psf2 = (torch.full((ny, nx), float("nan"), device="cuda") for _ in range(2))
        grad = torch.full(prob.h_shape, float("nan"), device="cuda")
        saved = torch.full((k, ny, nx), float("nan"), dtype=torch.complex64, device="cuda")

        def ws(op):
            got, nbytes = api.group_workspace_size(prob, op, group, op == L.DOP_OP_PSF)
            assert got == min(group, k)
            return torch.empty(nbytes, dtype=torch.uint8, device="cuda"), nbytes

        buf, n = ws(L.DOP_OP_PSF)
        L.check(L.lib().dop_psf(ctx.handle, prob.ptr(), ptr(h), ptr(a), ptr(psf), None, ptr(buf), n,
                                stream), "dop_psf")
        L.check(L.lib().dop_psf(ctx.handle, prob.ptr(), ptr(h), ptr(a), ptr(psf2), ptr(saved),
                                ptr(buf), n, stream), "dop_psf")
        buf, n = ws(L.DOP_OP_PSF_BACKWARD)
        L.check(L.lib().dop_psf_backward(ctx.handle, prob.ptr(), ptr(h), ptr(a), ptr(saved), ptr(g),
                                         ptr(grad), ptr(buf), n, stream), "dop_psf_backward")
        torch.cuda.synchronize()
        return psf, psf2, saved, grad

    one, grouped = calls(1), calls(4)
    for name, x, y in zip(("psf", "psf with saved fields", "saved fields", "gradient"), one, grouped):
        assert torch.equal(x, y), name
    assert torch.equal(one[0], one[1])
    table = np.ndim(m) > 0 or m & (m - 1)
    if table:
        for group in (1, 4):
            ctx.profile_enable(True)
            calls(group)
            count = ctx.profile_read()
            ctx.profile_enable(False)
            assert count["pass_a_fwd"][0] == count["pass_a_inv"][0] == 3 * -(-k // group)
