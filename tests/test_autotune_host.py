"""The autotuner's choice on the CPU: the planner and the tuner compiled with
g++ against the HIP stub, with a stand-in for the launch whose time is a rule
(tests/sanitize/tune_driver.cpp).  Where exec runs on tiles that no request
names, the planner's own choice has to be timed among the candidates, kept
where it wins, recorded, and found again from the record and from the reported
tile."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_1705_06661_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")

STAND_INS = ["hipEventCreate", "hipEventDestroy", "hipEventRecord", "hipEventSynchronize",
             "hipEventElapsedTime", "spinsum_exec"]


def test_autotune_keeps_the_planners_choice(tmp_path):
    base = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
            "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    rename = [f"-D{f}=stub_{f}" for f in STAND_INS]
    objs, procs = [], []
    for src, extra in ((os.path.join(CSRC, "spinsum_plan.cpp"), []),
                       (os.path.join(CSRC, "spinsum_tune.cpp"), []),
                       (os.path.join(SAN, "hip_host_stub.cpp"), rename),
                       (os.path.join(SAN, "tune_driver.cpp"), [])):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        procs.append(subprocess.Popen(base + extra + ["-c", src, "-o", objs[-1]],
                                      stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    for p in procs:
        out, _ = p.communicate(timeout=600)
        assert p.returncode == 0, out[-4000:]
    exe = str(tmp_path / "tune_driver")
    subprocess.run(["g++"] + objs + ["-o", exe], check=True, timeout=300)
    env = {k: v for k, v in os.environ.items() if k != "SPINSUM_AUTOTUNE_CACHE"}
    r = subprocess.run([exe, str(tmp_path)], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "PASSED" in r.stdout, r.stdout + r.stderr
    assert r.stdout.count("ok ") == 5
