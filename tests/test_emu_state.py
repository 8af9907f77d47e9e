"""What the C ABI's calls leave behind, on the CPU emulation of the device: queued work, allocations, device waits.

The emulator queues stream work and runs it at synchronisation points, so a test sees what is still pending when a call
returns.  Cases: tests/emu/run_state.py.
"""
import importlib.util
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
_BUILD = os.path.join(HERE, "emu", "build.py")
if not os.path.exists(_BUILD):
    pytest.skip("the emulation's sources are not here", allow_module_level=True)
_spec = importlib.util.spec_from_file_location("emu_build", _BUILD)
emu_build = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(emu_build)
pytestmark = pytest.mark.skipif(not emu_build.available(), reason="clang++ with the ASan runtime not found")


@pytest.fixture(scope="module")
def emu_lib():
    return emu_build.build()


def _run(lib, case):
    env = dict(os.environ, LD_PRELOAD=emu_build.asan_runtime(), ASAN_OPTIONS="detect_leaks=0:abort_on_error=1",
               EMU_STACK_KB="64", EMU_STRICT="1")
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_state.py"), lib, case], env=env,
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "ok  " in r.stdout and "FAIL" not in r.stdout, r.stdout[-4000:] + r.stderr[-4000:]


@pytest.mark.parametrize("case", ["krr_create", "adjoint_map", "own_device", "krr_lanes", "krr_failures",
                                  "noalloc_shares", "narrow_splits", "product_buffers", "adjoint_degree0",
                                  "factor_memory"])
def test_state_after_calls(emu_lib, case):
    _run(emu_lib, case)
