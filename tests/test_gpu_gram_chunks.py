"""The Gram passes where their chunks change from one tile of 16 points to four, against the oracle.

The first pass changes at 64 x 4,096 points, the refining one at that divided by the refined degrees.  Ranks are equal to
the oracle's and the binary64 product is within 1e-12, as in the parity tests.
"""
import numpy as np
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


CASES = [(262_080, 1.0, 1e-3, False), (262_081, 1.0, 1e-3, False), (262_145, 1.0, 1e-3, False),
         (15, 0.5, 1e-8, False), (20_033, 0.35, 1e-9, True), (66_575, 0.35, 1e-9, True)]


@pytest.mark.parametrize("n,l,tol,refined", CASES, ids=lambda v: str(v))
def test_chunk_edges(n, l, tol, refined):
    from paper_2202_03655_amd import hdf
    X = wl.unit_ball(n, 3, 900)
    st = ohdf.build(X, "gaussian", l, tol)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)
    assert f.info()["rank"] == st["r"]
    if refined:
        assert f.info()["n_refined"] > 1
    V = wl.rhs(n, 2, 901)
    assert rel_fro(f.matvec(to_dev(V, torch.float64)).cpu().numpy(), ohdf.matvec(st, V)) <= 1e-12
