"""The factor evaluation split over workgroups against one workgroup's worth of points evaluated unsplit.

The matrix-free chunk of a large cloud is not needed for this: the harmonics and radial functions of a point depend on
that point and the plan alone, so a factor of a cloud holds the same bits in every row however the launch is cut.  The
oracle's harmonics are the reference (relative to the largest of a row: 1e-12 in binary64, as in the parity test).
Sizes: one point, a wavefront's edge, more points than one workgroup, in every dimension, and degrees from 0 up.
"""
import numpy as np
import pytest
import torch

from oracle import hdf as ohdf
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import degree_blocks, oracle_phi, rel_fro, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d,n,l,tol", [(3, 1, 1.0, 1e-4), (3, 129, 0.5, 1e-6), (4, 513, 0.8, 1e-5), (5, 64, 1.5, 1e-4),
                                       (6, 1031, 2.0, 1e-4), (7, 300, 2.0, 1e-4), (8, 257, 2.0, 1e-3), (3, 700, 50.0, 1e-2)])
def test_split_evaluation(d, n, l, tol):
    from paper_2202_03655_amd import hdf
    X = wl.unit_ball(n, d, 600 + d)
    st = ohdf.build(X, "gaussian", l, tol)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)
    assert f.info()["rank"] == st["r"]
    phi, q = f.factor_parts()
    kept = [k for k, s in enumerate(f.info()["s_k"]) if s]
    ref = oracle_phi(st, kept)
    assert phi.shape == ref.shape
    assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-12 * max(1.0, np.abs(ref).max())
    V = wl.rhs(n, 3, 601)
    assert rel_fro(f.matvec(to_dev(V, torch.float64)).cpu().numpy(), ohdf.matvec(st, V)) <= 1e-12
    assert len(degree_blocks(f)) == len(kept) and q.shape[0] == f.info()["n_radial"]


def test_rows_do_not_depend_on_the_launch():
    """The first points of a large cloud (one or few groups) and the factor of matrix-free chunks (many groups) agree."""
    from paper_2202_03655_amd import hdf
    X = to_dev(wl.max_norm_one(wl.gaussian_mixture(60_011, 5, 103)), torch.float32)
    V = to_dev(wl.rhs(60_011, 4, 602), torch.float32)
    stored = hdf.Factor(X, "cauchy", 1.0, 1e-4).matvec(V)
    chunked = hdf.Factor(X, "cauchy", 1.0, 1e-4, storage="none", fused=False, chunk=1000).matvec(V)
    # the same factor values; the partial sums of the passes are cut differently (binary32 accumulators)
    assert rel_fro(chunked.double().cpu().numpy(), stored.double().cpu().numpy()) <= 1e-6
