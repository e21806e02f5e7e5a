"""The precision form's FP64 fallback over contiguous lines, every system of
the batch falling back (no refinement step): parity at the refined bar."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["shared", "shift", "perrow"])
@pytest.mark.parametrize("n,nsys", [(4, 1000), (16, 257), (64, 65), (100, 300), (720, 40), (1500, 9), (2000, 3)])
def test_every_contiguous_line_falls_back(kind, n, nsys):
    import paper_2509_03933_amd as tdma
    p = configs.partitioned(4, 4, n) if kind == "perrow" else configs.adi(4, 4, n)
    layout = configs.Layout(n=n, nsys0=nsys, row_stride=1, sys_stride0=n)
    p = dataclasses.replace(p, layout=layout, law="perrow" if kind == "perrow" else "uniform_d")
    if kind == "shift":
        p = dataclasses.replace(p, shift=np.linspace(0.0, 2.0, nsys))
    a, b, c, d = parity.host_problem(p)
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tx = torch.full_like(td, float("nan"))
    rep = tdma.solve_refined(p.layout, coeffs, td, tx, max_iters=0)
    tdma.check()
    assert rep["fallback_systems"] == rep["not_converged"] == nsys, rep
    err = parity.per_system_error(p.layout, tx.cpu().numpy(), ref)
    assert err.max() <= parity.TOL_REFINED, err.max()
