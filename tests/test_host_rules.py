"""Host rules of the library that need no GPU: launch sizes, plans and tables, checked in
a driver (tests/host/plan_checks.hip) that includes the runtime's source and links with the
built library."""
import os
import re
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


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="ROCm compilers not available")
def test_parts_meet_by_release_and_acquire(tmp_path):
    """In the code of the batched FP4 matcher, a part's minima are waited for before the workgroup's
    barrier, the count of finished parts is a release to the device, and the last part acquires
    before its second barrier, after which it reads the others' results."""
    asm = str(tmp_path / "knn.s")
    made = subprocess.run(
        [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-fno-honor-nans", "-I", os.path.join(ROOT, "include"), "-S",
         "--offload-device-only", os.path.join(PACKAGE, "csrc", "knn.hip"), "-o", asm],
        capture_output=True, text=True)
    assert made.returncode == 0, made.stdout + made.stderr
    text = open(asm).read()
    kernels = re.findall(r"^(_ZN\S*knn_batch_fp4_kernel\S*):.*?s_endpgm", text, re.S | re.M)
    assert len(kernels) == 2
    for body in re.findall(r"^_ZN\S*knn_batch_fp4_kernel\S*:(.*?)s_endpgm", text, re.S | re.M):
        marks = re.findall(r"(global_atomic_umin_x2|s_waitcnt vmcnt\(0\)|s_barrier|buffer_wbl2 sc1|"
                           r"global_atomic_add|buffer_inv sc1)", body)
        tail = " ".join(marks[len(marks) - 1 - marks[::-1].index("global_atomic_umin_x2"):])
        assert re.search(r"umin_x2 (s_waitcnt vmcnt\(0\) )+s_barrier (s_waitcnt vmcnt\(0\) )*buffer_wbl2 sc1 "
                         r"(s_waitcnt vmcnt\(0\) )*global_atomic_add (s_waitcnt vmcnt\(0\) )+buffer_inv sc1 "
                         r"(s_waitcnt vmcnt\(0\) )*s_barrier", tail), tail
