"""What the library's calls leave behind on the emulated device: queued work, allocations, waits.

Started in a subprocess with the ASan runtime preloaded (tests/test_emu_state.py):
    LD_PRELOAD=<libclang_rt.asan> python tests/emu/run_state.py <libhdf_emu.so> [case ...]
Unlike run_cases.py the library's calls are not followed by a flush unless a case asks for one, so the emulator's
counters are read as a caller on another stream would find them.
"""
import ctypes
import sys

import numpy as np
import torch

import run_cases as rc
from run_cases import _raw, check, dense, hdf, rel, to_dev, wl

_raw.emu_pending.restype = ctypes.c_longlong


def _krr(n=90, k=3, d=3, seed=31):
    X = wl.unit_ball(n, d, seed)
    lab = np.random.default_rng(seed).integers(0, k, n).astype(np.int32)
    S = hdf.KRR(to_dev(X, torch.float64), to_dev(lab, torch.int32), k, "gaussian", 0.8, 1e-6, 0.1)
    return X, S


def case_krr_create():
    """hdf_krr_create is blocking: nothing that the operator reads is still queued on its stream when it returns."""
    X, S = _krr()
    left = _raw.emu_pending()
    check("krr_create", left == 0, f"{left} operations still queued on return")
    v = wl.rhs(len(X), 1, 32)[:, 0]
    y = S.apply(to_dev(v, torch.float64))
    _raw.emu_flush()
    e = rel(y.numpy(), dense.dense_K(X, "gaussian", 0.8) @ v + 0.1 * v)
    check("krr_create apply", e <= 1e-6, f"{e:.2e}")


CASES = {"krr_create": case_krr_create}

if __name__ == "__main__":
    rc._install()
    hdf._lib = hdf._lib._L                       # no flush after the calls
    for name in (sys.argv[2:] or list(CASES)):
        CASES[name]()
    sys.exit(1 if check.failed else 0)
