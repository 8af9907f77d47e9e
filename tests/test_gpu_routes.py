"""Products that take the routes the other tests only come near, against references of their own.

Chunked matrix-free products of more than 64 columns: several slabs of 64 in one launch into the chunk scratch, binary32
and binary64, compared with the same columns in narrower products (bounds of the test of stored wide products).  Pass 2 on
the matrix cores over all blocks at once with more than eight radial functions per degree, one to four 16-column tiles per
wavefront: 65,501 points are 1,024 groups of 64, where groups of one, two, three and four tiles fill the 1,024 SIMDs
exactly once; binary64 against the oracle, 1e-12 as in the parity tests.
"""
import pytest
import torch

from oracle import hdf as ohdf
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import rel_fro, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("m", [65, 80, 128, 129, 193, 256])
@pytest.mark.parametrize("dt,bound", [(torch.float32, 1e-5), (torch.float64, 1e-12)], ids=["f32", "f64"])
def test_wide_chunked_product(dt, bound, m):
    from paper_2202_03655_amd import hdf
    n = 4_099
    prec = hdf.HDF_FP64 if dt == torch.float64 else hdf.HDF_MIXED
    f = hdf.Factor(to_dev(wl.unit_ball(n, 4, 821), dt), "gaussian", 1.0, 1e-4, precision=prec, storage="none", chunk=1500,
                   fused=False)
    assert f.info()["mf_fused"] == 0
    V = to_dev(wl.rhs(n, 300, 823), dt)[:, 7:7 + m]
    parts = torch.cat([f.matvec(V[:, c:c + 48]) for c in range(0, m, 48)], dim=1)
    assert rel_fro(f.matvec(V).cpu().numpy(), parts.cpu().numpy()) <= bound


def test_unsplit_pass2_many_radial_functions():
    from paper_2202_03655_amd import hdf
    n = 65_501
    X = wl.unit_ball(n, 3, 822)
    st = ohdf.build(X, "gaussian", 0.35, 1e-9)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", 0.35, 1e-9, precision=hdf.HDF_FP64)
    assert f.info()["rank"] == st["r"] and max(f.info()["s_k"]) > 8
    V = wl.rhs(n, 64, 824)
    ref = ohdf.matvec(st, V)
    for m in (5, 20, 33, 64):
        assert rel_fro(f.matvec(to_dev(V[:, :m], torch.float64)).cpu().numpy(), ref[:, :m]) <= 1e-12, m
