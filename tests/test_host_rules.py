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
def test_order_of_the_accesses_of_parts(tmp_path):
    """In the code of the batched FP4 matcher, a part's minima are waited for before the workgroup's
    barrier, the count of finished parts follows it, and the loads of the last part, which do not
    stop at the XCD's L2 (sc1), follow the next one."""
    asm = str(tmp_path / "knn.s")
    made = subprocess.run(
        [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-fno-honor-nans", "-I", os.path.join(ROOT, "include"), "-S",
         "--offload-device-only", os.path.join(PACKAGE, "csrc", "knn.hip"), "-o", asm],
        capture_output=True, text=True)
    assert made.returncode == 0, made.stdout + made.stderr
    kernels = re.findall(r"^_ZN\S*knn_batch_fp4_kernel\S*:(.*?)s_endpgm", open(asm).read(), re.S | re.M)
    assert len(kernels) == 2
    for body in kernels:
        marks = re.findall(r"(global_atomic_umin_x2|s_waitcnt vmcnt\(0\)|s_barrier|global_atomic_add|"
                           r"global_load_dwordx2 [^\n]*sc1)", body)
        marks = ["load sc1" if m.startswith("global_load") else m for m in marks]
        tail = " ".join(marks[len(marks) - 1 - marks[::-1].index("global_atomic_umin_x2"):])
        wait = r"(s_waitcnt vmcnt\(0\) )"
        assert re.search("umin_x2 " + wait + "+s_barrier " + wait + "*global_atomic_add " + wait +
                         "+s_barrier " + wait + "*load sc1 (load sc1|s_waitcnt vmcnt)", tail), tail
