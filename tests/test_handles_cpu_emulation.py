"""Handles of matrices in pair form under the host emulation of the kernels
with AddressSanitizer (cpu_hip/handles.cpp), one check per test."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def unit():
    sys.path.insert(0, os.path.join(HERE, "cpu_hip"))
    import build_cpu
    build_cpu.build()
    exe = os.path.join(build_cpu.OUT_DIR, "handles")
    objs = [os.path.join(build_cpu.OUT_DIR, s.replace(".hip", ".o")) for s in build_cpu.SOURCES]
    subprocess.run(["g++"] + build_cpu.FLAGS + [os.path.join(HERE, "cpu_hip", "handles.cpp"),
                                                "-x", "none"] + objs + ["-o", exe], check=True)
    return exe


CHECKS = ["failed_reassembly", "left_pair_form"]


@pytest.mark.parametrize("check", CHECKS)
def test_handles(unit, check):
    r = subprocess.run([unit, check], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and "all ok" in r.stdout, r.stdout[-3000:] + r.stderr[-3000:]
