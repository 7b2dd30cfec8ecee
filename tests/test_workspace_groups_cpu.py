"""dop_workspace_size_group on the CPU: how many wavelengths an operation runs
together and the workspace that takes.  A half-filled plane on 4096 .. 16384,
3600^2 there, and grids whose passes do not group get one field however many
wavelengths there are; asking for less than the limit gives that."""

import ctypes

import numpy as np
import pytest

from paper_2505_22313_amd import _lib as L
from paper_2505_22313_amd import api


def problem(m, n, k, mode="crop", up=1):
    return api.Problem(n, m, 0.5, 900.0, np.linspace(0.45, 0.65, k), [1.46] * k, out_mode=mode,
                       upsample=up)


def field(m):
    my, mx = (m, m) if np.ndim(m) == 0 else m
    return 8 * my * (mx + 16)


# grid, DOE, window, wavelengths run together of 6: PSF, PSF with saved
# fields, gradient
CASES = [
    (1024, 512, "crop", 4, 4, 4), (2048, 2048, "crop", 4, 4, 4), (16, 3, "full", 4, 1, 1),
    (4096, 2048, "crop", 1, 1, 1), (8192, 4096, "crop", 1, 1, 1), (16384, 100, "crop", 1, 1, 1),
    (4096, 2049, "crop", 4, 1, 1), (8192, 4096, "full", 4, 1, 1), (32768, 16384, "crop", 4, 1, 1),
    (3072, 1536, "crop", 4, 1, 1), (3600, 1800, "crop", 1, 1, 1), (3600, 1801, "crop", 1, 1, 1),
    (3600, 2700, "crop", 4, 1, 1), (2144, 1072, "crop", 1, 1, 1), (720, 360, "crop", 4, 4, 4),
    ((240, 2144), (120, 1072), "crop", 1, 1, 1), ((16080, 10720), (8040, 5360), "crop", 1, 1, 1),
    ((5360, 240), (2680, 120), "crop", 4, 4, 4),
]


@pytest.mark.parametrize("m,n,mode,psf,saved,grad", CASES)
def test_group_and_bytes(m, n, mode, psf, saved, grad):
    p = problem(m, n, 6, mode)
    assert api.group_workspace_size(p, L.DOP_OP_PSF) == (psf, psf * field(m))
    assert api.group_workspace_size(p, L.DOP_OP_PROPAGATE) == (1, field(m))
    assert api.workspace_size(p) == field(m)
    if mode == "crop":
        assert api.group_workspace_size(p, L.DOP_OP_PSF, 4, True) == (saved, saved * field(m))
        assert api.group_workspace_size(p, L.DOP_OP_PSF_BACKWARD) == (grad, grad * field(m))
    for want in (1, 2, 3, 9):
        g = min(want, psf)
        assert api.group_workspace_size(p, L.DOP_OP_PSF, want) == (g, g * field(m))
    few = problem(m, n, 2, mode)
    g = min(psf, 2)
    if not (np.ndim(m) == 0 and m == 3600):  # (there the passes depend on the count)
        assert api.group_workspace_size(few, L.DOP_OP_PSF) == (g, g * field(m))


def test_gradient_of_a_coarse_design_has_its_fine_map_behind_the_fields():
    p = problem(240, 120, 3, up=4)
    fields = -(-3 * field(240) // 256) * 256
    assert api.group_workspace_size(p, L.DOP_OP_PSF_BACKWARD) == (3, fields + 4 * 120 * 120)


def test_arguments():
    p = problem(1024, 512, 3)
    g, b = ctypes.c_int(0), ctypes.c_size_t(7)
    fn = L.lib().dop_workspace_size_group
    assert fn(None, p.ptr(), L.DOP_OP_PSF, 0, ctypes.byref(g), ctypes.byref(b)) == L.DOP_ERR_INVALID_ARG
    assert fn(None, p.ptr(), L.DOP_OP_PSF, 0, None, ctypes.byref(b)) == L.DOP_ERR_INVALID_ARG
    assert fn(None, p.ptr(), L.DOP_OP_PSF, 0, ctypes.byref(g), None) == L.DOP_ERR_INVALID_ARG
    g.value = 4
    assert fn(None, p.ptr(), 9, 0, ctypes.byref(g), ctypes.byref(b)) == L.DOP_ERR_INVALID_ARG
    assert fn(None, None, L.DOP_OP_PSF, 0, ctypes.byref(g), ctypes.byref(b)) == L.DOP_ERR_INVALID_ARG
    assert g.value == 4 and b.value == 7


class _Context:
    """Stands for api.Context where the memory holds `most` bytes."""

    device = 0

    def __init__(self, most):
        self.most, self.group_cap, self.asked = most, {}, []

    def workspace(self, nbytes, stream):
        self.asked.append(nbytes)
        if nbytes > self.most:
            raise api.torch.cuda.OutOfMemoryError("out of memory")
        return object()


def test_binding_falls_back_to_fewer_fields_and_remembers():
    p = problem(1024, 512, 6)
    f = field(1024)
    ctx = _Context(2 * f)
    assert api._workspace(ctx, p, L.DOP_OP_PSF, 0)[1] == 2 * f
    assert ctx.asked == [4 * f, 3 * f, 2 * f]
    assert api._workspace(ctx, p, L.DOP_OP_PSF_BACKWARD, 0)[1] == 2 * f
    assert api._workspace(ctx, p, L.DOP_OP_PSF, 0, group=1)[1] == f
    assert ctx.asked[3:] == [2 * f, f]
    ctx = _Context(f - 1)
    with pytest.raises(api.torch.cuda.OutOfMemoryError):
        api._workspace(ctx, p, L.DOP_OP_PSF, 0)
    assert ctx.asked[-1] == f
