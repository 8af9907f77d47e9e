"""The preconditioner's block inverses at the edges of their 64-wide tiles, against a dense binary64 solve.

Clusters of one point, of one tile and its neighbours, and of several tiles with a remainder in one system.  The bound is
that of the preconditioner's parity test: the blocks' condition is at most (n + lambda) / lambda < 5e3, and a backward
stable solve of n < 400 unknowns is within about n * condition * 1e-16 < 1e-9 in the worst case, 1e-10 in practice.
"""
import numpy as np
import pytest
import torch

from oracle import dense
from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import rel_fro, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes", [(1,), (63, 64, 65), (1, 127, 128, 129, 2), (331, 5, 192)], ids=str)
def test_inverse_at_tile_edges(sizes):
    from paper_2202_03655_amd import hdf
    n = sum(sizes)
    X = wl.unit_ball(n, 3, 500 + n)
    lab = np.random.default_rng(n).permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    S = hdf.KRR(to_dev(X, torch.float64), to_dev(lab, torch.int32), len(sizes), "gaussian", 0.8, 1e-4, 0.1)
    r = wl.rhs(n, 1, 501)[:, 0]
    z = S.precond(to_dev(r, torch.float64)).cpu().numpy()
    for c in range(len(sizes)):
        at = np.flatnonzero(lab == c)
        A = dense.dense_K(X[at], "gaussian", 0.8)
        ref = np.linalg.solve(A + 0.1 * np.eye(len(at)), r[at])
        assert rel_fro(z[at], ref) <= 1e-10


def test_singular_block_is_refused():
    """Identical points and a vanishing lambda: the second pivot of the block is exactly zero."""
    from paper_2202_03655_amd import hdf
    X = np.full((70, 3), 0.25)
    with pytest.raises(hdf.HDFError, match=r"cluster 0 is not positive definite \(pivot 2\)"):
        hdf.KRR(to_dev(X, torch.float64), torch.zeros(70, dtype=torch.int32, device="cuda"), 1, "gaussian", 1.0, 1e-4,
                1e-300)
