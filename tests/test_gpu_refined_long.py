"""GPU parity of the precision form at the longest strided lines of a shared
operator that its on-chip state holds (16 rows per lane, one system per tile),
and the refusal of the next length."""
import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [5729, 5800, 5840])
def test_longest_strided_lines(n):
    import paper_2509_03933_amd as tdma
    p = configs.adi(6, 3, n)
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_refined(p.layout, coeffs, td, tx)
    tdma.check()
    ref = parity.oracle_solution(p, a, b, c, d)
    err = parity.per_system_error(p.layout, tx.cpu().numpy(), ref)
    assert err.max() <= parity.TOL_REFINED, err.max()


def test_next_length_is_refused():
    import paper_2509_03933_amd as tdma
    p = configs.adi(6, 3, 5841)
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    with pytest.raises(tdma.TdmaError) as ei:
        tdma.solve_refined(p.layout, coeffs, td, torch.empty_like(td))
    assert ei.value.status == tdma.EUNSUPPORTED
