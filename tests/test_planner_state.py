"""What the host planner keeps for the process, under sanitizers (g++, host code only): tests/native/planner_state_main.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", params=["address,undefined", "thread"])
def exe(request, tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("planner") / "planner_state"
    csrc = os.path.join(ROOT, "paper_2202_03655_amd", "csrc")
    r = subprocess.run([gxx, "-O1", "-g", "-std=c++17", f"-fsanitize={request.param}", "-fno-sanitize-recover", "-I", csrc,
                        os.path.join(ROOT, "tests", "native", "planner_state_main.cpp"),
                        os.path.join(csrc, "planner.cpp"), "-o", str(out), "-lpthread"],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return str(out)


@pytest.mark.parametrize("case", ["maps", "pools"])
def test_kept_state(exe, case):
    r = subprocess.run([exe, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout
