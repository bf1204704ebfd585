"""The stop flag of the PCG loop under the host emulation of the kernels with
AddressSanitizer (cpu_hip/stop_flag.cpp): blocks that start while block 0 of
their launch sets the flag change no row, and solves that converge and solves
that break down (p.Ap < 0) give the same bits whether every block combines the
partials itself or a one-block kernel does."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_stop_flag_is_uniform_over_a_block():
    sys.path.insert(0, os.path.join(HERE, "cpu_hip"))
    import build_cpu
    build_cpu.build()
    objs = [os.path.join(build_cpu.OUT_DIR, s.replace(".hip", ".o"))
            for s in build_cpu.SOURCES if s != "solve.hip"]
    # one order of additions in both builds: no second level of the reductions
    flags = [f for f in build_cpu.FLAGS if not f.startswith("-DRT_PARTIAL_FOLD_MIN")]
    exes = {f: os.path.join(build_cpu.OUT_DIR, f"stop_flag_{f}") for f in (4096, 0)}
    builds = [subprocess.Popen(["g++"] + flags + [f"-DRT_FUSED_PARTIALS={f}",
                                                  os.path.join(HERE, "cpu_hip", "stop_flag.cpp"),
                                                  "-x", "none"] + objs + ["-o", exe])
              for f, exe in exes.items()]
    assert [p.wait() for p in builds] == [0, 0]
    lines = []
    for exe in exes.values():
        r = subprocess.run([exe], capture_output=True, text=True, timeout=900,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert r.returncode == 0 and "all ok" in r.stdout, r.stdout[-3000:] + r.stderr[-3000:]
        lines.append([s for s in r.stdout.splitlines() if s.startswith("solve ")])
    assert len(lines[0]) == 4 and lines[0] == lines[1]
