"""Pass 2 at the edges of its column groups, block shares and harmonic batches, against the oracle.

A wavefront takes one to four 16-column tiles, so right-hand-side counts around every group edge are tried, in binary64
(1e-12 as in the parity tests), with enough points for one launch over all blocks (> 64 x 1,024), with few points (blocks
in shares, also more shares than a degree has blocks) and with more than eight radial functions per degree (two runs over
a degree's rows).
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


CASES = [
    # n, d, l, tol, right-hand sides
    (66_001, 3, 1.0, 1e-4, (1, 16, 17, 33, 49, 80, 129, 200)),
    (1_337, 4, 0.9, 1e-5, (1, 31, 64, 65, 113, 256)),
    (97, 8, 2.0, 1e-3, (1, 48)),
    (2_003, 3, 0.35, 1e-9, (3, 20)),
    (70_001, 3, 0.35, 1e-9, (2,)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}_d{c[1]}_l{c[2]}")
def test_column_groups_and_shares(case):
    from paper_2202_03655_amd import hdf
    n, d, l, tol, ms = case
    X = wl.unit_ball(n, d, 700 + d)
    st = ohdf.build(X, "gaussian", l, tol)
    f = hdf.Factor(to_dev(X, torch.float64), "gaussian", l, tol, precision=hdf.HDF_FP64)
    assert f.info()["rank"] == st["r"]
    if l < 0.5:
        assert max(f.info()["s_k"]) > 8
    V = wl.rhs(n, max(ms), 701)
    ref = ohdf.matvec(st, V)
    for m in ms:
        Vd = to_dev(V[:, :m], torch.float64)
        assert rel_fro(f.matvec(Vd).cpu().numpy(), ref[:, :m]) <= 1e-12, m
        if m <= 64:
            out = torch.full((n, m + 3), float("nan"), dtype=torch.float64, device="cuda")[:, :m]
            assert rel_fro(f.matvec_noalloc(Vd, out).cpu().numpy(), ref[:, :m]) <= 1e-12, m
