"""A KRR system made on one stream and used on others, without an ordering by the caller: hdf_krr_create is blocking.

The first use of each kind reads what construction left last (descriptors of the batched products, zeroed entries of
rank-zero factors).  Against the dense operator, bound as in the tests of the concurrent builds.
"""
import numpy as np
import pytest
import torch

from oracle import dense
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(300, 1), (1_501, 12)])
def test_first_use_on_another_stream(n, k):
    from paper_2202_03655_amd import hdf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X = wl.unit_ball(n, 3, 640 + k)
    lab = to_dev(np.random.default_rng(k).integers(0, k, n).astype(np.int32), torch.int32)
    Xd, v = to_dev(X, torch.float64), to_dev(wl.rhs(n, 1, 641)[:, 0], torch.float64)
    torch.cuda.synchronize()
    made, used = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(made):
        S = hdf.KRR(Xd, lab, k, "gaussian", 0.8, 1e-8, 0.1)
    with torch.cuda.stream(used):
        y = S.apply(v)
    used.synchronize()
    K = dense.dense_K(X, "gaussian", 0.8)
    vh = v.cpu().numpy()
    assert np.linalg.norm(y.cpu().numpy() - (K @ vh + 0.1 * vh)) <= 1e-8 * np.linalg.norm(K) * np.linalg.norm(vh)
