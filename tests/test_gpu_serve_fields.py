"""Workspace that the chunked server holds for a request: as many fields as the
request's wavelength groups can use.  A half-filled plane on 4096^2 runs one
wavelength at a time and holds one field; a whole plane there runs groups of
four and holds four; the results are dop_psf's, bitwise."""

import numpy as np
import pytest

from paper_2505_22313_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_22313_amd import api as _api
    yield _api
    _api.default_context(0).release_workspaces()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("m,n,mode,fields", [
    (4096, 2048, "crop", 1), (4096, 2048, "full", 4), (4096, 2049, "crop", 4),
    (3600, 1800, "crop", 1), (3600, 1801, "crop", 1), (3600, 2700, "crop", 4),
    (1024, 512, "crop", 4), (2144, 1072, "crop", 1),
])
def test_request_holds_the_fields_it_uses(api, m, n, mode, fields):
    lams = np.linspace(0.45, 0.65, 6)
    prob = api.Problem(n, m, 0.5, 900.0, lams, wl.cauchy_index(lams), out_mode=mode)
    h = torch.from_numpy(wl.uniform_heights(n, seed=m + n)).cuda()
    alone = api.psf(h, prob)
    out = torch.full(prob.out_shape, float("nan"), device="cuda")
    torch.cuda.synchronize()
    field = -(-api.workspace_size(prob) // 256) * 256
    srv = api.Server(9 * field, max_slots=2)
    try:
        srv.wait(srv.submit(prob, h, out), 60.0)
        assert srv.stats()["arena_peak"] == fields * field
    finally:
        srv.close()
    assert torch.equal(alone, out)
