"""The launch plan of a batched pass, on the CPU: tests/plan_driver.hip is compiled with the library's
host source and linked with the other objects of the normal build."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.timeout(600)
def test_plan_without_products(tmp_path):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("hipcc not available")
    from paper_1503_07037_amd import build as B
    objs = [os.path.join(B.BUILD_DIR, s.replace(".hip", ".o")) for s in B.SOURCES if s != "dmpt_api.hip"]
    if not all(os.path.exists(o) for o in objs):
        B.build()
    obj, exe = str(tmp_path / "plan_driver.o"), str(tmp_path / "plan_driver")
    flags = ["-O1" if f == "-O3" else f for f in B.FLAGS]
    B._run([B._hipcc(), *flags, "-c", os.path.join(ROOT, "tests", "plan_driver.hip"), "-o", obj])
    B._run([B._hipcc(), f"--offload-arch={B.ARCH}", obj, *objs, *B.LINK, "-o", exe])
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    print(p.stdout[-2000:])
    assert p.returncode == 0 and "plan driver: ok" in p.stdout
