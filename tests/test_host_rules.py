"""Host rules of the library that need no GPU: launch sizes, plans and tables, checked in
a driver (tests/host/plan_checks.hip) that includes the runtime's source and links with the
built library."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1609_03986_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PACKAGE = os.path.join(ROOT, "paper_1609_03986_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="ROCm compilers not available")
def test_host_rules(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    obj, exe = str(tmp_path / "plan_checks.o"), str(tmp_path / "plan_checks")
    compile_it = [HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature",
                  "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-c",
                  os.path.join(HERE, "host", "plan_checks.hip"), "-o", obj]
    link_it = [HIPCC, "--offload-arch=gfx950", obj, build.LIB,
               "-Wl,-rpath," + PACKAGE, "-o", exe]
    for cmd in (compile_it, link_it):
        made = subprocess.run(cmd, capture_output=True, text=True)
        assert made.returncode == 0, made.stdout + made.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr


@pytest.fixture(scope="module")
def matcher_code(tmp_path_factory):
    """The assembly of the matchers' kernels by name, as the library is built."""
    if not os.path.exists(HIPCC):
        pytest.skip("ROCm compilers not available")
    asm = str(tmp_path_factory.mktemp("asm") / "knn.s")
    made = subprocess.run(
        [HIPCC] + build.HIPCC_FLAGS + build.FILE_FLAGS["knn.hip"] +
        ["-I", os.path.join(ROOT, "include"), "-S", "--offload-device-only",
         os.path.join(PACKAGE, "csrc", "knn.hip"), "-o", asm], capture_output=True, text=True)
    assert made.returncode == 0, made.stdout + made.stderr
    return dict(re.findall(r"^(_ZN\S*):(.*?)s_endpgm", open(asm).read(), re.S | re.M))


def test_order_of_the_accesses_of_parts(matcher_code):
    """In the code of the batched FP4 matcher, a part's minima are waited for before the workgroup's
    barrier, the count of finished parts follows it, and the loads of the last part, which do not
    stop at the XCD's L2 (sc1), follow the next one."""
    kernels = [code for name, code in matcher_code.items() if "knn_batch_fp4_kernel" in name]
    assert len(kernels) == 2
    for body in kernels:
        marks = re.findall(r"(global_atomic_umin_x2|s_waitcnt vmcnt\(0\)|s_barrier|global_atomic_add|"
                           r"global_load_dwordx2 [^\n]*sc1)", body)
        marks = ["load sc1" if m.startswith("global_load") else m for m in marks]
        tail = " ".join(marks[len(marks) - 1 - marks[::-1].index("global_atomic_umin_x2"):])
        wait = r"(s_waitcnt vmcnt\(0\) )"
        assert re.search("umin_x2 " + wait + "+s_barrier " + wait + "*global_atomic_add " + wait +
                         "+s_barrier " + wait + "*load sc1 (load sc1|s_waitcnt vmcnt)", tail), tail


@pytest.mark.parametrize("kernel", ["knn_popcount_kernel", "knn_batch_popcount_kernel"])
def test_train_rows_come_through_scalar_loads(matcher_code, kernel):
    """The popcount matchers read a train row, which is uniform over a wavefront, with scalar loads:
    the 16-byte vector loads are the query's row alone."""
    code = next(code for name, code in matcher_code.items() if kernel in name)
    assert code.count("s_load_dwordx16") >= 4
    assert code.count("global_load_dwordx4") == 4
