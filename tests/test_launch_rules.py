"""The rules by which the host picks kernels and divides work, called through the library's own functions.  No GPU needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_08358_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not available")


def _run(tmp_path, body):
    """Compiles a main() around `body` against the library's headers and library, runs it and returns what it prints."""
    src, exe, lib = tmp_path / "rules.hip", tmp_path / "rules", os.path.dirname(CSRC)
    src.write_text('#include <stdio.h>\n#include "mar_split.h"\nint main() {\n' + body + "\nreturn 0;\n}\n")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe), "-L", lib,
                        "-lmarius_hip", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split()


def test_one_workgroup_sorts_less_where_nothing_runs_beside_it(tmp_path):
    """One workgroup takes longer over 9,000 to 16,384 rows than the launches it replaces: in the pipeline and above 256 floats,
    where its own time counts, half as many rows."""
    out = _run(tmp_path, """for (int alone = 0; alone < 2; ++alone) for (int dk : {16, 256, 260, 400}) printf("%d ", mar_sort_one_limit(dk, alone));""")
    assert [int(x) for x in out] == [16384, 16384, 8192, 8192] + [8192] * 4
