"""The counter summary that bench.py reports HBM traffic from (CPU only): a
record written by the profiling tool is one that bench.py accepts, for its own
grid and no other."""

import importlib.util
import json
import os
import subprocess
import sys

import pytest

from paper_2505_22313_amd import profiling as pr
from test_host_tools_cpu import ROOT, write_counters

COPY = pr.CALIB_KERNEL
KIB = 4 * 1024 ** 3 / 1024


@pytest.fixture
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def write_run(path, plans=(16,)):
    rows = [("void dop::k_pass_c<%d>(dop::KParams)" % p, c, 1000.0) for p in plans
            for c in ("FETCH_SIZE", "WRITE_SIZE")]
    for sub, c in (("fetch", "FETCH_SIZE"), ("write", "WRITE_SIZE")):
        write_counters(path / sub, [(COPY, c, KIB)] + [r for r in rows if r[1] == c])
    return str(path / "fetch"), str(path / "write")


def test_record_of_the_tool_is_reported(tmp_path, bench, monkeypatch):
    fetch, write = write_run(tmp_path)
    out = subprocess.run([sys.executable, "-m", "paper_2505_22313_amd.profiling", "traffic", fetch,
                          write, "32768"], cwd=ROOT, check=True, capture_output=True, text=True)
    rec = json.loads(out.stdout)
    assert rec["m"] == 65536 and rec["n"] == 32768 and rec["command"] and rec["calibration"]
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "traffic_large_65536.json").write_text(out.stdout)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.measured_traffic("pass_c", 65536) == 2 * 1000 * 1024
    assert bench.measured_traffic("pass_c", 32768) is None


def test_counters_of_one_grid_only(tmp_path):
    with pytest.raises(RuntimeError):
        pr.traffic(*write_run(tmp_path / "two", plans=(15, 16)))
    with pytest.raises(RuntimeError):
        pr.traffic(*write_run(tmp_path / "table", plans=(105,)))


def test_source_hash_covers_what_the_kernels_include(tmp_path, monkeypatch):
    """The hash follows the includes of the pass kernels' source: a change in
    any of these files makes a recorded figure stale."""
    names = {os.path.basename(p) for p in pr.kernel_sources()}
    assert {"asm_kernels.hip", "asm_device.h", "asm_stages.h", "dop_internal.h"} <= names
    files = {"a.hip": '#include <x.h>\n#include "b.h"\nint a;\n', "b.h": '  # include "sub/c.h"\n',
             "sub/c.h": '#include "../b.h"\nint c;\n', "other.h": "int o;\n"}
    (tmp_path / "sub").mkdir()
    for name, text in files.items():
        (tmp_path / name).write_text(text)
    monkeypatch.setattr(pr.kernel_sources, "__defaults__", (str(tmp_path / "a.hip"),))
    first = pr.kernel_source_hash()
    (tmp_path / "other.h").write_text("int p;\n")
    assert pr.kernel_source_hash() == first
    for name in ("a.hip", "b.h", "sub/c.h"):
        text = (tmp_path / name).read_text()
        (tmp_path / name).write_text(text + "int more;\n")
        assert pr.kernel_source_hash() != first
        (tmp_path / name).write_text(text)
