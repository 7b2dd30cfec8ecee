"""Which passes an operation takes (CPU only): tests/c/route_check.cpp asks the
library's own rule for each problem below."""

import os
import shutil
import subprocess

import pytest

from paper_2505_22313_amd import _lib as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(ROCM + "/include/hip"):
        pytest.skip("no host C++ compiler or no HIP headers")
    if not os.path.exists(L.LIB_PATH):
        pytest.skip("libdop.so not built")
    exe = str(tmp_path_factory.mktemp("c") / "route_check")
    subprocess.run([gxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", ROCM + "/include",
                    os.path.join(ROOT, "tests", "c", "route_check.cpp"), L.LIB_PATH,
                    "-L", ROCM + "/lib", "-lamdhip64",
                    "-Wl,-rpath," + os.path.dirname(L.LIB_PATH) + ":" + ROCM + "/lib", "-o", exe],
                   check=True)

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True)
        return dict(line.split() for line in out.stdout.splitlines())

    return run


@pytest.mark.parametrize("my,mx,ny,nx,k,full,psf,field,gradient", [
    # square powers of two and the table grids that fit: one rule for all
    (1024, 1024, 700, 512, 3, 0, "small", "small", "small"),
    (2048, 2048, 2048, 2048, 1, 1, "small", "small", "small"),
    (240, 2144, 200, 2000, 4, 1, "small", "small", "small"),
    # half-filled planes, and what is just over half or wants the whole plane
    (4096, 4096, 2048, 2048, 3, 0, "tri", "tri", "tri"),
    (4096, 4096, 2049, 2048, 3, 0, "five", "five", "five"),
    (16384, 16384, 8192, 8193, 1, 0, "five", "five", "five"),
    (8192, 8192, 4096, 4096, 1, 1, "five", "five", "five"),
    (32768, 32768, 16384, 16384, 1, 0, "five", "five", "five"),
    (3072, 3072, 1536, 1536, 4, 0, "five", "five", "five"),
    # 3600^2: by the rows of the first and last pass, and the wavelengths
    (3600, 3600, 1800, 1800, 4, 0, "tri", "tri", "tri"),
    (3600, 3600, 2700, 2700, 1, 0, "small", "small", "small"),
    (3600, 3600, 2701, 2700, 1, 0, "five", "five", "small"),
    (3600, 3600, 2000, 2700, 4, 0, "small", "small", "small"),
    (3600, 3600, 2001, 2700, 4, 0, "five", "small", "small"),
    (3600, 3600, 400, 1800, 4, 1, "small", "small", "small"),
    (3600, 3600, 1800, 1800, 1, 1, "small", "small", "small"),
    (3600, 3600, 1800, 1800, 2, 1, "five", "small", "small"),
    (3600, 3600, 1801, 1800, 1, 1, "five", "five", "small"),
])
def test_route(check, my, mx, ny, nx, k, full, psf, field, gradient):
    got = check(my, mx, ny, nx, k, full)
    assert (got["psf"], got["field"], got["gradient"]) == (psf, field, gradient)


def test_three_pass_launcher_refuses_what_its_kernels_do_not_run(check):
    """A group of wavelengths (its kernels would skip all but the first) and
    problems outside the half planes, before anything is launched."""
    got = check("refuse")
    assert got and all(v == "1" for v in got.values()), got
