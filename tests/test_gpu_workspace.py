"""The workspace that the binding keeps for a stream: one field where an
operation runs one wavelength at a time, the group's where it groups, and the
group a caller asks for at most."""

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


@pytest.mark.parametrize("m,n,psf,saved,grad", [
    (4096, 2048, 1, 1, 1), (4096, 2049, 4, 1, 1), (8192, 4096, 1, 1, 1), (2144, 1072, 1, 1, 1),
    (1024, 512, 4, 4, 4), (3600, 1801, 1, 1, 1),
])
def test_kept_workspace(api, m, n, psf, saved, grad):
    lams = np.linspace(0.45, 0.65, 5)
    prob = api.Problem(n, m, 0.5, 900.0, lams, wl.cauchy_index(lams))
    h = torch.from_numpy(wl.uniform_heights(n, seed=m + n)).cuda()
    ctx = api.Context(0)
    stream = torch.cuda.current_stream(0).cuda_stream
    field = api.workspace_size(prob)

    def kept(fn):
        ctx.release_workspaces()
        out = fn()
        fields, rest = divmod(ctx.workspace_bytes(stream), field)
        assert rest == 0
        return out, fields

    out, fields = kept(lambda: api.psf(h, prob, ctx=ctx))
    assert fields == psf
    one, fields = kept(lambda: api.psf(h, prob, ctx=ctx, group=1))
    assert fields == 1 and torch.equal(out, one)
    (again, u), fields = kept(lambda: api.psf(h, prob, ctx=ctx, save_fields=True))
    assert fields == saved and torch.equal(out, again)
    _, fields = kept(lambda: api.psf_backward(h, prob, u, out, ctx=ctx))
    assert fields == grad
    ctx.close()
