"""Products of more than 64 right-hand sides, which pass 1 takes in slabs of 64 columns.

Columns are independent, so a wide product is compared with the same columns in narrower ones.  The two differ in the
split of the points and the order of the sums only: binary64 agrees to 1e-12; in binary32 a sum of up to a few thousand
terms in a row is within about sqrt(4,000) x 6e-8 = 4e-6 of its value, bound 1e-5.
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


KINDS = [("stored_f32", torch.float32, 1e-5), ("stored_f64", torch.float64, 1e-12), ("cross_f32", torch.float32, 1e-5),
         ("chunked_f32", torch.float32, 1e-5), ("binary64_factor", torch.float32, 1e-5)]


@pytest.mark.parametrize("m", [65, 80, 128, 129, 193, 256])
@pytest.mark.parametrize("kind", KINDS, ids=lambda c: c[0])
def test_wide_product(kind, m):
    from paper_2202_03655_amd import hdf
    name, dt, bound = kind
    n = 4_099
    X = to_dev(wl.unit_ball(n, 4, 811), dt)
    prec = hdf.HDF_FP64 if dt == torch.float64 else hdf.HDF_MIXED
    if name == "cross_f32":
        f = hdf.CrossFactor(to_dev(wl.unit_ball(333, 4, 812), dt), X, "gaussian", 1.0, 1e-4, precision=prec)
    elif name == "chunked_f32":
        f = hdf.Factor(X, "gaussian", 1.0, 1e-4, precision=prec, storage="none", chunk=1500)
    else:
        f = hdf.Factor(X, "gaussian", 1.0, 1e-8 if name == "binary64_factor" else 1e-4, precision=prec)
    V = to_dev(wl.rhs(n, 300, 813), dt)[:, 7:7 + m]               # rows further apart than the columns
    wide = f.matvec(V)
    parts = torch.cat([f.matvec(V[:, c:c + 48]) for c in range(0, m, 48)], dim=1)
    assert rel_fro(wide.cpu().numpy(), parts.cpu().numpy()) <= bound
