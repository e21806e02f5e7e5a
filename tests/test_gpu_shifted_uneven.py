"""GPU parity of the shifted-operator plan (FP64, strided) on batches past the
small-batch rule: lengths whose partitions leave one to four row slots empty,
fill them, or go to the generic kernel; in place.  The operator is diagonally
dominant (ADI tables and positive shifts); the tolerance is the parity bar."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [40, 64, 200, 256, 257, 301, 400, 511, 512, 545, 640, 700, 897, 1000, 1023, 1100, 2000])
def test_uneven_shifted_lines(n):
    import paper_2509_03933_amd as tdma
    n0 = 67
    n1 = -(-3200000 // (n0 * n))
    p = configs.adi(n0, n1, n)
    p = dataclasses.replace(p, shift=np.linspace(0.0, 3.0, n0 * n1))
    a, b, c, d = parity.host_problem(p)
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.cpu().numpy(), ref)
    assert err.max() <= parity.TOL_F64, err.max()
    tdma.solve_batched(p.layout, coeffs, td, td)
    assert torch.equal(td, tx)


def test_kernel_7_explicit_tiles_keep_their_rule():
    """An explicit kernel 7 tile needs 16 or 32 rows per lane and P*M = n."""
    import paper_2509_03933_amd as tdma
    p = configs.adi(8, 8, 640)
    p = dataclasses.replace(p, shift=np.ones(64))
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    for M, P in ((20, 32), (32, 32), (24, 32)):
        with pytest.raises(tdma.TdmaError) as ei:
            tdma.solve_batched_tiled(p.layout, coeffs, td, torch.empty_like(td), M=M, S=8, P=P, kernel=7)
        assert ei.value.status == tdma.EINVAL
