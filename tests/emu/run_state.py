"""What the library's calls leave behind on the emulated device: queued work, allocations, waits.

Started in a subprocess with the ASan runtime preloaded (tests/test_emu_state.py):
    LD_PRELOAD=<libclang_rt.asan> python tests/emu/run_state.py <libhdf_emu.so> [case ...]
Unlike run_cases.py the library's calls are not followed by a flush unless a case asks for one, so the emulator's
counters are read as a caller on another stream would find them.
"""
import ctypes
import os
import sys

import numpy as np
import torch

import run_cases as rc
from run_cases import _raw, check, dense, hdf, rel, to_dev, wl

for _f in ("emu_pending", "emu_mallocs", "emu_frees", "emu_waits", "emu_launching_threads", "emu_launches", "emu_memsets", "emu_live"):
    getattr(_raw, _f).restype = ctypes.c_longlong


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


def _ball_factor(l, tol, n=24):
    return hdf.Factor(to_dev(wl.unit_ball(n, 3, 33), torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)


def _degree(f):
    s_k = f.info()["s_k"]
    assert all(s_k[:len(s_k)]) or s_k.index(0) == len([x for x in s_k if x]), "kept degrees are 0..K"
    return sum(1 for x in s_k if x) - 1


def _dx(f, n=24):
    W, V = (to_dev(wl.rhs(n, 1, s), torch.float64) for s in (34, 35))
    g = f.backward(W, V, need_l=False)[1]
    _raw.emu_flush()
    return g.numpy().copy()


def case_adjoint_map():
    """A factor keeps the derivative map that its enqueued work reads: factors of nine other degrees, then another of its
    own degree, come between two of its gradients, and the second gives back no memory."""
    first = _ball_factor(1.0, 1e-4)
    g1, K = _dx(first), _degree(first)
    seen = {K}
    for tol in (1e-1, 1e-2, 1e-3, 1e-5, 1e-6, 1e-7, 1e-8, 1e-10, 1e-11):
        for l in (0.8, 1.0, 1.6):
            f = _ball_factor(l, tol)
            if _degree(f) not in seen and len(seen) < 10:
                seen.add(_degree(f))
                _dx(f)
    check("adjoint_map degrees", len(seen) == 10, f"{sorted(seen)}")
    other = _ball_factor(1.0, 1e-4)
    _dx(other)
    before = _raw.emu_frees()
    g2 = _dx(first)
    freed = _raw.emu_frees() - before
    check("adjoint_map kept", freed == 0, f"{freed} buffers given back while work may read them")
    check("adjoint_map gradient", np.array_equal(g1, g2), "the same bits again")


def case_own_device():
    """What is freed while another device is current waits for its own device."""
    for what in ("factor", "krr"):
        _raw.hipSetDevice(1)
        obj = _ball_factor(1.0, 1e-4) if what == "factor" else _krr()[1]
        _raw.hipSetDevice(0)
        before = _raw.emu_waits(0), _raw.emu_waits(1)
        del obj
        now = _raw.emu_waits(0), _raw.emu_waits(1)
        check(f"own_device {what}", now[1] > before[1] and now[0] == before[0],
              f"waits for devices 0 and 1: {before} before, {now} after")
        dev = ctypes.c_int(-1)
        _raw.hipGetDevice(ctypes.byref(dev))
        check(f"own_device {what} current", dev.value == 0, f"device {dev.value} is current")


def case_krr_lanes():
    """The concurrent block builds of a KRR system run here too (several host threads launch kernels), and the operator
    is that of the dense system."""
    before = _raw.emu_launching_threads()
    X, S = _krr(n=1100, k=24, seed=37)
    threads = _raw.emu_launching_threads() - before
    check("krr_lanes threads", threads >= 2 or (os.cpu_count() or 1) < 2, f"{threads} more threads launched kernels")
    v = wl.rhs(len(X), 1, 32)[:, 0]
    y = S.apply(to_dev(v, torch.float64))
    _raw.emu_flush()
    e = rel(y.numpy(), dense.dense_K(X, "gaussian", 0.8) @ v + 0.1 * v)
    check("krr_lanes apply", e <= 1e-6, f"{e:.2e}")


def _status(make):
    try:
        return 0, make()
    except hdf.HDFError as e:
        return e.status, str(e)


def case_krr_failures():
    """A block build that fails beside others: for want of memory it is repeated alone, any other failure is reported
    once, and an infeasible build is not made twice."""
    _raw.emu_fail(0, 20)                         # construction's own allocations before the builds: 6
    st, made = _status(_krr)
    check("krr_failures memory", st == 0, f"status {st}")
    if st == 0:
        X, S = made
        v = wl.rhs(len(X), 1, 32)[:, 0]
        y = S.apply(to_dev(v, torch.float64))
        _raw.emu_flush()
        e = rel(y.numpy(), dense.dense_K(X, "gaussian", 0.8) @ v + 0.1 * v)
        check("krr_failures memory apply", e <= 1e-6, f"{e:.2e}")
    _raw.emu_fail(1, 8)                          # and its own copies: 6
    st, msg = _status(_krr)
    _raw.emu_fail(1, 0)
    check("krr_failures copy", st == -6 and "factor of cluster" in str(msg), f"status {st}: {msg}")
    X = to_dev(wl.unit_ball(90, 3, 31), torch.float64)
    n0 = _raw.emu_launches()
    st, _ = _status(lambda: hdf.Factor(X, "gaussian", 1e-3, 1e-6, precision=hdf.HDF_FP64))
    n1 = _raw.emu_launches()
    sk, msg = _status(lambda: hdf.KRR(X, to_dev(np.zeros(90, np.int32), torch.int32), 1, "gaussian", 1e-3, 1e-6, 0.1))
    n2 = _raw.emu_launches()
    check("krr_failures infeasible", st == sk == -4 and n2 - n1 < 2 * (n1 - n0),
          f"status {st}, {sk}; {n1 - n0} launches of a build, {n2 - n1} of the construction")


def case_noalloc_shares():
    """hdf_matvec_noalloc splits pass 2 of few points and few right-hand sides as hdf_matvec does, the shares in its
    fixed scratch (one launch more than without a split), and both give the same bits."""
    n = 700
    f = hdf.Factor(to_dev(wl.unit_ball(n, 4, 36), torch.float64), "gaussian", 1.0, 1e-4, precision=hdf.HDF_FP64)
    for m in (1, 4):
        V, out = to_dev(wl.rhs(n, m, 37), torch.float64), rc.dev_empty((n, m), torch.float64)
        counts = []
        def noalloc():
            assert hdf.lib().hdf_matvec_noalloc(f._h, V.data_ptr(), m, m, out.data_ptr(), m, None) == 0
            return out
        for run in (lambda: f.matvec(V), noalloc):
            _raw.emu_flush()
            before = _raw.emu_launches()
            ref = run()
            _raw.emu_flush()
            counts.append((_raw.emu_launches() - before, ref.numpy().copy()))
        check(f"noalloc_shares m={m}", counts[0][0] == counts[1][0] and np.array_equal(counts[0][1], counts[1][1]),
              f"{counts[0][0]} and {counts[1][0]} launches")


def case_narrow_splits():
    """Pass 1 of a narrow product of a thousand binary32 points runs in two splits (one launch more, their sum)."""
    for n, launches in ((511, 3), (1100, 4)):
        X = wl.unit_ball(n, 3, 38).astype(np.float32)
        f = hdf.Factor(to_dev(X, torch.float32), "gaussian", 1.0, 1e-3, precision=hdf.HDF_MIXED)
        V = wl.rhs(n, 4, 39).astype(np.float32)
        Vd = to_dev(V, torch.float32)
        _raw.emu_flush()
        before = _raw.emu_launches()
        y = f.matvec(Vd)
        _raw.emu_flush()
        count = _raw.emu_launches() - before
        e = rel(y.numpy().astype(np.float64), rc.ohdf.matvec(rc.ohdf.build(X.astype(np.float64), "gaussian", 1.0, 1e-3), V))
        check(f"narrow_splits n={n}", count == launches and e <= 1e-5, f"{count} launches, {e:.2e}")


def case_product_buffers():
    """After one product of a stored factor, others allocate nothing: any of up to 16 right-hand sides with many points,
    those of no more right-hand sides with few (whose pass 2 is split), and those of the same 16 columns."""
    few, many = range(1, 17), (1, 2, 3, 4, 5, 16)
    for n, tol, first, then in ((700, 1e-4, 16, few), (700, 1e-4, 8, range(1, 9)), (700, 1e-4, 4, range(1, 5)),
                                (66_000, 0.3, 1, many), (66_000, 0.3, 5, many), (50_000, 0.3, 20, (32, 17, 16, 3))):
        f = _ball_factor(1.0, tol, n)
        V = wl.rhs(n, max(first, *then), 40)
        f.matvec(to_dev(V[:, :first], torch.float64))
        before = _raw.emu_mallocs()
        for m in then:
            f.matvec(to_dev(V[:, :m], torch.float64))
        more = _raw.emu_mallocs() - before
        check(f"product_buffers n={n} first {first}", more == 0, f"{more} allocations by the products of {list(then)}")
        _raw.emu_flush()


def case_adjoint_degree0():
    """dF/dX of a factor of degree 0 alone: no memset nodes in what may be captured, and the oracle's gradient."""
    n = 40
    X = wl.unit_ball(n, 3, 41)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", 50.0, 0.5, precision=hdf.HDF_FP64)
    W, V = wl.rhs(n, 3, 42), wl.rhs(n, 3, 43)
    _raw.emu_flush()
    before = _raw.emu_memsets()
    g = f.backward(to_dev(W, torch.float64), to_dev(V, torch.float64), need_l=False)[1]
    _raw.emu_flush()
    sets = _raw.emu_memsets() - before
    st = rc.ohdf.build(X, "gaussian", 50.0, 0.5)
    e = rel(g.numpy(), rc.ohdf.grad_x(st, W, V))
    check("adjoint_degree0", _degree(f) == 0 and sets == 0 and e <= 1e-10, f"s_k {f.info()['s_k']}, {sets} memsets, {e:.2e}")


def case_factor_memory():
    """A built factor holds its rows, the points and tables, not the records of the Gram pass (1.3 MB for these points)."""
    n = 5000
    X, Y = (to_dev(wl.unit_ball(m, 3, 44), torch.float64) for m in (n, 300))
    for what in ("symmetric", "general"):
        before = _raw.emu_live()
        f = hdf.Factor(X, "gaussian", 1.0, 1e-4, precision=hdf.HDF_FP64) if what == "symmetric" else \
            hdf.CrossFactor(Y, X, "gaussian", 1.0, 1e-4, precision=hdf.HDF_FP64)
        _raw.emu_flush()
        rest = _raw.emu_live() - before - f.info()["factor_bytes"]
        check(f"factor_memory {what}", rest <= 600_000, f"{rest} bytes beside the rows")
        del f


CASES = {"factor_memory": case_factor_memory, "adjoint_degree0": case_adjoint_degree0, "product_buffers": case_product_buffers, "narrow_splits": case_narrow_splits, "noalloc_shares": case_noalloc_shares, "krr_failures": case_krr_failures, "krr_lanes": case_krr_lanes, "own_device": case_own_device, "adjoint_map": case_adjoint_map, "krr_create": case_krr_create}

if __name__ == "__main__":
    rc._install()
    hdf._lib = hdf._lib._L                       # no flush after the calls
    for name in (sys.argv[2:] or list(CASES)):
        CASES[name]()
    sys.exit(1 if check.failed else 0)
