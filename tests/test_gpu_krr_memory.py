"""Device memory of a KRR system: large blocks go back to the device, where other libraries can have them."""
import numpy as np
import pytest
import torch

from paper_2202_03655_amd import workloads as wl
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


def test_large_blocks_are_given_back():
    from paper_2202_03655_amd import hdf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 8192                                              # one cluster: inverse and work storage of 512 MiB each

    def system(m):
        return hdf.KRR(to_dev(wl.unit_ball(m, 3, 660), torch.float64), to_dev(np.zeros(m, np.int32), torch.int32), 1,
                       "gaussian", 1.0, 1e-6, 0.1)

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0] / 2**20
    system(500)                                           # loads the kernels
    before = free()
    S = system(n)
    held = before - free()
    y = S.apply(to_dev(wl.rhs(n, 1, 661)[:, 0], torch.float64))
    assert torch.isfinite(y).all()
    del S, y
    left = before - free()
    # the factor (38 rows), vectors and 27 partial sums of 8,192 points and the build's records: below 100 MiB
    assert held <= 512 + 100, held
    assert left <= 100, left
