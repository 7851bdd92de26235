"""Host rules of the library that need no GPU: launch sizes, plans and tables, checked in
a driver (tests/host/plan_checks.hip) that includes the runtime's source and links with the
built library."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PACKAGE = os.path.join(ROOT, "paper_1609_03986_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="ROCm compilers not available")
def test_host_rules(tmp_path):
    obj, exe = str(tmp_path / "plan_checks.o"), str(tmp_path / "plan_checks")
    compile_it = [HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature",
                  "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-c",
                  os.path.join(HERE, "host", "plan_checks.hip"), "-o", obj]
    link_it = [HIPCC, "--offload-arch=gfx950", obj, os.path.join(PACKAGE, "liblatch.so"),
               "-Wl,-rpath," + PACKAGE, "-o", exe]
    for cmd in (compile_it, link_it):
        made = subprocess.run(cmd, capture_output=True, text=True)
        assert made.returncode == 0, made.stdout + made.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
