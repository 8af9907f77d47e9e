"""Products with one to five right-hand sides: the narrow passes (up to four) and the matrix-core passes next to them.

Against the oracle in binary64 (1e-12, the parity tests' bound) and, for binary32, against an independent binary64
contraction of the same stored factor (4e-6, the bound of the parity test of that kind).  Sizes: one point, a wavefront's
points (128 binary64, 256 binary32) and their neighbours, several splits; a strided V and output; degrees with more than
four radial functions.
"""
import pytest
import torch

from oracle import hdf as ohdf
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import gpu_build, rel_fro, to_dev, torch_contraction

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,d,l,tol", [(1, 3, 1.0, 1e-4), (127, 3, 0.5, 1e-6), (128, 4, 1.0, 1e-4), (129, 5, 1.5, 1e-4),
                                       (40_003, 3, 0.4, 1e-8), (9_001, 4, 0.8, 1e-6), (700, 8, 2.0, 1e-3)])
def test_narrow_binary64(n, d, l, tol):
    from paper_2202_03655_amd import hdf
    X = wl.unit_ball(n, d, 800 + d)
    st = ohdf.build(X, "gaussian", l, tol)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)
    V = wl.rhs(n, 9, 801)
    ref = ohdf.matvec(st, V)
    Vd = to_dev(V, torch.float64)
    for m in (1, 2, 3, 4, 5):
        wide = torch.full((n, m + 2), float("nan"), dtype=torch.float64, device="cuda")
        f.matvec(Vd[:, 2:2 + m], out=wide[:, :m])
        assert rel_fro(wide[:, :m].cpu().numpy(), ref[:, 2:2 + m]) <= 1e-12, m
        assert torch.isnan(wide[:, m:]).all()
        out = torch.empty((n, m), dtype=torch.float64, device="cuda")
        assert rel_fro(f.matvec_noalloc(Vd[:, 2:2 + m], out).cpu().numpy(), ref[:, 2:2 + m]) <= 1e-12, m


@pytest.mark.parametrize("n", [255, 256, 12_037])
def test_narrow_binary32(n):
    X = wl.max_norm_one(wl.gaussian_mixture(n, 5, 103)).astype("float32")
    f, _ = gpu_build(X, "cauchy", 1.0, 1e-4, mixed=True)
    for m in (1, 2, 3, 4, 5):
        V = to_dev(wl.rhs(n, m, 802 + m).astype("float32"), torch.float32)
        assert rel_fro(f.matvec(V).double().cpu().numpy(), torch_contraction(f, V).cpu().numpy()) <= 4e-6, m


def test_narrow_cross_and_data_type():
    """The Y side of a general factor, and a binary64 factor of binary32 data."""
    from paper_2202_03655_amd import hdf
    X, Y = wl.unit_ball(333, 3, 803), wl.unit_ball(20_011, 3, 804)
    f = hdf.CrossFactor(to_dev(X, torch.float64), to_dev(Y, torch.float64), "gaussian", 0.8, 1e-6)
    px, qx = f.factor_parts()
    py, qy = f.factor_parts_y()
    W = to_dev(wl.rhs(20_011, 2, 805), torch.float64)
    ref, h0, q0 = torch.zeros(333, 2, dtype=torch.float64, device="cuda"), 0, 0
    for k, s in enumerate(f.info()["s_k"]):
        if not s:
            continue
        nh = 2 * k + 1
        for j in range(s):
            ux, uy = px[h0:h0 + nh] * qx[q0 + j], py[h0:h0 + nh] * qy[q0 + j]
            ref += ux.t().contiguous() @ (uy @ W)
        h0, q0 = h0 + nh, q0 + s
    assert rel_fro(f.matvec(W).cpu().numpy(), ref.cpu().numpy()) <= 1e-12
    X = wl.shell(3_001, 6, 105).astype("float32")
    g, _ = gpu_build(X, "matern52", 8.0, 1e-7, mixed=True)
    V = to_dev(wl.rhs(3_001, 3, 806).astype("float32"), torch.float32)
    # the output is rounded to binary32
    assert rel_fro(g.matvec(V).double().cpu().numpy(), torch_contraction(g, V).cpu().numpy()) <= 2e-7
