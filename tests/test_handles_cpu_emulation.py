"""Handles of matrices in pair form (cpu_hip/handles.cpp, one check per test),
the offsets of its external columns (cpu_hip/pair_scan.cpp) and plain shapes on
batches of them (cpu_hip/batch_shape.cpp) under the host emulation of the
kernels with AddressSanitizer."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _build(name, without=()):
    """A C++ unit linked with the library's sources (without those it includes)."""
    import build_cpu
    exe = os.path.join(build_cpu.OUT_DIR, name)
    objs = [os.path.join(build_cpu.OUT_DIR, s.replace(".hip", ".o")) for s in build_cpu.SOURCES
            if s not in without]
    subprocess.run(["g++"] + build_cpu.FLAGS + [os.path.join(HERE, "cpu_hip", name + ".cpp"),
                                                "-x", "none"] + objs + ["-o", exe], check=True)
    return exe


def _run(*cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout[-3000:] + r.stderr[-3000:]


@pytest.fixture(scope="module")
def library():
    sys.path.insert(0, os.path.join(HERE, "cpu_hip"))
    import build_cpu
    build_cpu.build()


@pytest.fixture(scope="module")
def unit(library):
    return _build("handles")


CHECKS = ["failed_reassembly", "left_pair_form", "left_untiled", "export_reads", "batch_reads",
          "tiles"]


@pytest.mark.parametrize("check", CHECKS)
def test_handles(unit, check):
    _run(unit, check)


def test_external_columns_past_32_bits(library):
    _run(_build("pair_scan", without=["pair.hip"]))


def test_plain_shape_of_a_batch(library):
    _run(_build("batch_shape", without=["batch.hip"]))
