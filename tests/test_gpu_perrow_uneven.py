"""GPU parity of the per-row plan on strided lines whose length no tile
divides (partitions of floor(n/P) and floor(n/P) + 1 rows in 16 to 32 row
slots), large enough to pass the small-batch rule: full slots, one to four
slots short, lengths below the kernel's range, both precisions, in place."""
import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [4, 20, 28, 33, 40, 100, 301, 480, 512, 545, 700, 897, 1000, 1025, 2000])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_uneven_lines(n, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = configs.partitioned(61, -(-1600000 // (61 * n)), n)
    a, b, c, d = parity.host_problem(p)
    if dtype == np.float32:
        a, b, c, d = [v.astype(np.float32).astype(np.float64) for v in (a, b, c, d)]
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    tol = parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32
    assert err.max() <= tol, err.max()
    tdma.solve_batched(p.layout, coeffs, td, td)
    assert torch.equal(td, tx)


def test_singular_pivot_in_uneven_partition():
    """A zero pivot in a partition's last row slot is flagged; slots that hold
    no row are not."""
    import paper_2509_03933_amd as tdma
    p = configs.partitioned(61, 27, 1000)
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tdma.solve_batched(p.layout, coeffs, td, torch.empty_like(td))
    tdma.check()
    for k in ("a", "b", "c"):
        coeffs[k].view(1000, -1)[999, 5] = 0.0
    tdma.solve_batched(p.layout, coeffs, td, torch.empty_like(td))
    with pytest.raises(tdma.TdmaError):
        tdma.check()
