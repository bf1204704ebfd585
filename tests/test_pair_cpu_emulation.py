"""The pair form of the fine level under the host emulation of the kernels
with AddressSanitizer (see test_kernels_cpu_emulation.py): structure, values,
products, steps and CSR rows on demand against the oracle.  The default run
takes one tile and a single particle; RT_CPU_FULL=1 runs every case."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ASAN = "/usr/lib/gcc/x86_64-linux-gnu/11/libasan.so"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(ASAN),
                    reason="needs g++ and libasan")
def test_pair_form_under_asan_matches_oracle():
    sys.path.insert(0, os.path.join(HERE, "cpu_hip"))
    import build_cpu
    env = dict(os.environ)
    env.update(RT_CPU_LIB=build_cpu.build(), LD_PRELOAD=ASAN,
               ASAN_OPTIONS="detect_leaks=0:max_malloc_fill_size=2147483647:malloc_fill_byte=190")
    if os.environ.get("RT_CPU_FULL") != "1":
        env.update(RT_CPU_CASES="mms2d_9,infinite3d_1", RT_CPU_QUICK="1")
    r = subprocess.run([sys.executable, "-u", os.path.join(HERE, "cpu_hip", "run_pair_cases.py")],
                       env=env, capture_output=True, text=True, timeout=3600)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-6000:]
    assert "all cases ok" in r.stdout
