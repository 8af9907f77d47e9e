"""Block factors built at the same time: fewer blocks than lanes, as many, more, and two callers at once.

The operator is compared with the dense one.  A block's factor is within tol of its kernel matrix in the Frobenius norm,
and what is outside the blocks is exact to rounding, so the product is within tol |K|_F |v|.
"""
import threading

import numpy as np
import pytest
import torch

from oracle import dense
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _system(n, k, seed):
    X = wl.unit_ball(n, 3, seed)
    lab = np.random.default_rng(seed).integers(0, k, n).astype(np.int32)
    lab[lab == 1] = 0                                     # cluster 1 stays empty where there is one
    return X, lab


@pytest.mark.parametrize("k", [1, 3, 9, 10, 11, 40])
def test_concurrent_builds(k):
    from paper_2202_03655_amd import hdf
    cases = [_system(700, k, 600 + k), _system(431, k, 700 + k)]
    out = [None, None]

    def fit(i):
        X, lab = cases[i]
        v = to_dev(wl.rhs(len(X), 1, 601)[:, 0], torch.float64)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(s):
            S = hdf.KRR(to_dev(X, torch.float64), to_dev(lab, torch.int32), k, "gaussian", 0.8, 1e-8, 0.1)
            y = S.apply(v)
        s.synchronize()
        out[i] = (v.cpu().numpy(), y.cpu().numpy())

    threads = [threading.Thread(target=fit, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for (X, lab), (v, y) in zip(cases, out):
        K = dense.dense_K(X, "gaussian", 0.8)
        assert np.linalg.norm(y - (K @ v + 0.1 * v)) <= 1e-8 * np.linalg.norm(K) * np.linalg.norm(v)


def test_first_failing_cluster_is_named():
    from paper_2202_03655_amd import hdf
    X, lab = _system(500, 12, 620)
    for c in (9, 4):
        X[np.flatnonzero(lab == c)[0], 1] = np.nan
    with pytest.raises(hdf.HDFError, match="factor of cluster 4: ") as e:
        hdf.KRR(to_dev(X, torch.float64), to_dev(lab, torch.int32), 12, "gaussian", 0.8, 1e-6, 0.1)
    assert e.value.status == -3
