"""Plain fused matrix-free kernels with one and with two slot groups, against the stored factor.

The factors' harmonics are too many for the double-buffered kernels (H = 1,210 ... 1,716) and their ranks around the slots
of one workgroup (192 row tiles, 768 steps).  Both products contract the same values in binary32 in other orders: a sum of
a few thousand terms is within about sqrt(4,000) x 6e-8 = 4e-6 of its value, bound 1e-5.
"""
import pytest
import torch

from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import rel_fro, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n", [600, 1_009, 20_011])
@pytest.mark.parametrize("d,l,tol", [(5, 0.6, 1e-4), (5, 0.55, 1e-4), (5, 0.6, 1e-5), (4, 0.4, 1e-5)], ids=str)
def test_slot_groups(d, l, tol, n):
    from paper_2202_03655_amd import hdf
    X = to_dev(wl.unit_ball(n, d, 5), torch.float32)
    f = hdf.Factor(X, "gaussian", l, tol, precision=hdf.HDF_MIXED, storage="none")
    assert f.info()["mf_fused"] >= 1                     # 2 where a degree less is kept: l = 0.6, 1e-4 at 20,011 points
    stored = hdf.Factor(X, "gaussian", l, tol, precision=hdf.HDF_MIXED)
    for m in (1, 16, 37):
        V = to_dev(wl.rhs(n, m, 951), torch.float32)
        assert rel_fro(f.matvec(V).cpu().numpy(), stored.matvec(V).cpu().numpy()) <= 1e-5, m
