"""The five digit passes on grids and DOEs that take no other path.

Gradients: against the FP64 oracle (1e-4, as everywhere) on 3072^2 and 4096^2,
with DOEs inside and over half the grid, an aperture, the fused upsampling, the
band limit and several wavelengths; on larger grids against the same chain put
together from dop_propagate (whose input and output stages share nothing with
the gradient's) and element-wise torch arithmetic: g_U = 2 w_k G U_k propagated
by -z, times conj(E_k).

Wavelength groups: bitwise what one wavelength at a time gives, over partial
groups, an aperture, the fused upsampling, the band limit, ragged DOEs and the
full window; the launch counts of a timed call show the groups."""

import os

import numpy as np
import pytest

import oracle
from oracle import asm
from paper_2505_22313_amd import workloads as wl
from _close import GRAD_ELEM, INTENSITY_ELEM, assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

asm.WORKERS = min(16, os.cpu_count() or 1)


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_22313_amd import api as _api
    return _api


@pytest.fixture(autouse=True)
def give_back(api):
    yield
    api.default_context(0).release_workspaces()
    torch.cuda.empty_cache()


def wavelengths(k):
    lams = np.linspace(0.42, 0.68, k) if k > 1 else np.array([0.55])
    return lams, np.linspace(0.5, 1.5, k).astype(np.float32)


def launches(api, fn):
    ctx = api.default_context(0)
    ctx.profile_enable(True)
    try:
        fn()
        return {name: v[0] for name, v in ctx.profile_read().items()}
    finally:
        ctx.profile_enable(False)


@pytest.mark.parametrize("m,ny,nx,k,up,amp,bl", [
    (3072, 1200, 1003, 2, 1, True, False), (3072, 2999, 3071, 3, 1, False, False),
    (3072, 1536, 1536, 2, 4, True, False), (3072, 700, 3072, 2, 2, False, True),
    (4096, 2052, 2056, 2, 4, True, False),
    (4096, 4095, 2049, 1, 1, True, True),
])
def test_gradient_matches_oracle(api, m, ny, nx, k, up, amp, bl):
    rng = np.random.default_rng(m + ny + nx + k)
    lams, w = wavelengths(k)
    nidx = wl.cauchy_index(lams)
    prob = api.Problem((ny, nx), m, 0.5, 800.0, lams, nidx, weights=w, upsample=up, bandlimit=bl)
    hc = rng.uniform(0.0, 1.2, prob.h_shape).astype(np.float32)
    a = rng.uniform(0.3, 1.0, (ny, nx)).astype(np.float32) if amp else None
    g = rng.standard_normal((ny, nx)).astype(np.float32)
    h, gd = torch.from_numpy(hc).cuda(), torch.from_numpy(g).cuda()
    ad = None if a is None else torch.from_numpy(a).cuda()
    _, fields = api.psf(h, prob, amp=ad, save_fields=True)
    grad = api.psf_backward(h, prob, fields, gd, amp=ad)
    count = launches(api, lambda: api.psf_backward(h, prob, fields, gd, amp=ad))
    assert count["pass_b_fwd"] == k
    hf = np.repeat(np.repeat(hc, up, axis=0), up, axis=1)
    want = oracle.psf_backward(hf, 0.5, 800.0, m, lams, nidx, g, weights=w, amp=a, bandlimit=bl)
    want = want.reshape(ny // up, up, nx // up, up).sum((1, 3))
    assert_close(grad, want, 1e-4, GRAD_ELEM, "gradient")


@pytest.mark.parametrize("m,ny,nx,k,up,amp", [
    (28800, 14400, 14400, 1, 8, False), (28800, 9001, 14399, 2, 1, True),
    (28800, 15001, 28800, 1, 1, True), (40000, 20000, 19996, 2, 4, True),
    ((16080, 10720), 8040, 5360, 2, 1, True), ((16080, 10720), 16080, 10712, 1, 4, False),
    ((16080, 10720), 3, 9001, 1, 1, False), (16384, 8200, 16383, 1, 1, True),
    (32768, 16384, 16384, 2, 1, False), (65536, 4001, 32768, 1, 1, True),
])
def test_gradient_matches_the_propagated_chain(api, m, ny, nx, k, up, amp):
    gen = torch.Generator(device="cuda").manual_seed(ny + nx + k)
    lams, w = wavelengths(k)
    nidx = wl.cauchy_index(lams)
    z = 900.0
    prob = api.Problem((ny, nx), m, 0.5, z, lams, nidx, weights=w, upsample=up)
    back = api.Problem((ny, nx), m, 0.5, -z, lams, nidx)
    h = torch.rand(prob.h_shape, generator=gen, device="cuda") * 1.2
    a = torch.rand((ny, nx), generator=gen, device="cuda") * 0.7 + 0.3 if amp else None
    g = torch.randn((ny, nx), generator=gen, device="cuda")
    _, fields = api.psf(h, prob, amp=a, save_fields=True)
    got = api.psf_backward(h, prob, fields, g, amp=a)
    want = torch.zeros((ny, nx), device="cuda")
    for i in range(k):
        ge = api.propagate(fields[i] * (2.0 * float(w[i]) * g), back, k=i)
        turns = (nidx[i] - 1.0) / lams[i]
        for r in range(0, ny, 4096):
            e = min(ny, r + 4096)
            q = turns * h[r // up:-(-e // up)].double()
            if up > 1:
                q = q.repeat_interleave(up, 0)[r % up:r % up + e - r].repeat_interleave(up, 1)
            q = (q - torch.round(q)).float() * (2.0 * np.pi)
            amps = 1.0 if a is None else a[r:e]
            want[r:e] += 2.0 * np.pi * turns * amps * (ge[r:e].imag * torch.cos(q)
                                                       - ge[r:e].real * torch.sin(q))
        del ge
    if up > 1:
        want = want.view(ny // up, up, nx // up, up).sum((1, 3))
    d = (got - want).abs()
    l2 = float(torch.linalg.vector_norm(d) / torch.linalg.vector_norm(want))
    el = float(d.max() / want.abs().max())
    assert l2 <= 1e-4 and el <= GRAD_ELEM, f"rel-L2 {l2:.2e}, element {el:.2e}"


@pytest.mark.parametrize("m,ny,nx,k,mode,up,amp,bl", [
    (3072, 1536, 1536, 2, "crop", 1, False, False), (3072, 1533, 1001, 7, "crop", 1, True, False),
    (3072, 2900, 3068, 4, "full", 4, True, False), (3072, 5, 3071, 5, "full", 1, False, True),
    (4096, 2049, 100, 3, "crop", 1, True, False), (4096, 2048, 2048, 6, "full", 2, False, False),
    (8192, 4097, 4096, 5, "crop", 1, True, True), (28800, 3001, 14400, 2, "crop", 1, True, False),
    (32768, 16384, 1000, 4, "crop", 8, True, False),
])
def test_groups_are_bitwise_one_wavelength_at_a_time(api, m, ny, nx, k, mode, up, amp, bl):
    rng = np.random.default_rng(m + ny + k)
    lams, w = wavelengths(k)
    nidx = wl.cauchy_index(lams)
    prob = api.Problem((ny, nx), m, 0.5, 900.0, lams, nidx, weights=w, out_mode=mode, upsample=up,
                       bandlimit=bl)
    hc = rng.uniform(0.0, 1.2, prob.h_shape).astype(np.float32)
    a = rng.uniform(0.3, 1.0, (ny, nx)).astype(np.float32) if amp else None
    h = torch.from_numpy(hc).cuda()
    ad = None if a is None else torch.from_numpy(a).cuda()
    one = api.psf(h, prob, amp=ad, group=1)
    grouped = api.psf(h, prob, amp=ad)
    assert torch.equal(one, grouped)
    for group in (1, 4):
        count = launches(api, lambda: api.psf(h, prob, amp=ad, group=group))
        assert count["pass_a_fwd"] == count["pass_a_inv"] == -(-k // group)
        assert count["pass_b_fwd"] == count["pass_c"] == count["pass_b_inv"] == k
    if m <= 4096:
        hf = np.repeat(np.repeat(hc, up, axis=0), up, axis=1)
        want = oracle.psf(hf, 0.5, 900.0, m, lams, nidx, weights=w, amp=a, out_mode=mode,
                          bandlimit=bl)
        assert_close(grouped, want, 2e-5, INTENSITY_ELEM, "psf")
