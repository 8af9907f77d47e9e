"""dF/dX and dF/dl with several columns are the sums of the columns' own.

F = sum_c w_c^T K~ v_c is linear in the pairs (w_c, v_c), so the gradients of a call with m columns equal the sums of m calls
with one: one column takes the narrow passes for both its contractions, two the narrow pass 1 and 2 for the radial part,
three and more the matrix-core passes, and 2 m > 256 two separate passes.  Binary64 rounding only (1e-12 of the largest
entry).  Degree 0 alone and the largest dimension are among the cases.
"""
import numpy as np
import pytest
import torch

from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,d,l,tol,ms", [(1_501, 3, 0.7, 1e-6, (2, 3, 9)), (611, 4, 1.0, 1e-4, (2, 130)),
                                          (300, 8, 2.0, 1e-3, (3,)), (257, 3, 300.0, 0.3, (1, 2, 3))])
def test_columns_add_up(n, d, l, tol, ms):
    from paper_2202_03655_amd import hdf
    X = wl.unit_ball(n, d, 900 + d)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)
    if l > 100:
        assert f.info()["degree_p"] == 0
    W, V = wl.rhs(n, max(ms), 901), wl.rhs(n, max(ms), 902)
    one = [f.backward(to_dev(W[:, c:c + 1], torch.float64), to_dev(V[:, c:c + 1], torch.float64)) for c in range(max(ms))]
    for m in ms:
        dl, dX = f.backward(to_dev(W[:, :m], torch.float64), to_dev(V[:, :m], torch.float64))
        refX = sum(o[1] for o in one[:m]).cpu().numpy()
        refl = sum(o[0] for o in one[:m])
        scale = max(float(np.abs(o[1].cpu().numpy()).max()) for o in one[:m]) * m
        assert np.abs(dX.cpu().numpy() - refX).max() <= 1e-12 * max(scale, 1e-300), m
        assert abs(dl - refl) <= 1e-12 * max(sum(abs(o[0]) for o in one[:m]), 1e-300) * 10, m
        assert f.backward(to_dev(W[:, :m], torch.float64), to_dev(V[:, :m], torch.float64), need_l=False)[0] is None
