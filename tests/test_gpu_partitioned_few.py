"""GPU parity of the staged solve of few contiguous lines, on both sides of the
numbers of systems from which every row's factors are kept (64 and 160 with
per-row coefficients in FP32 and FP64, 768 of a shared operator, 1,280 with a
shift), in one batch and in several.  Tolerances are the parity bars."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode,dtype,edge", [("perrow", np.float32, 64), ("perrow", np.float64, 160),
                                             ("shared", np.float32, 768), ("shared", np.float64, 768),
                                             ("shift", np.float32, 1280), ("shift", np.float64, 1280)])
@pytest.mark.parametrize("side", [-1, 0, 1])
@pytest.mark.parametrize("n", [79, 300, 1001])
def test_few_contiguous_lines(mode, dtype, edge, side, n):
    import paper_2509_03933_amd as tdma
    nsys = edge + side
    layout = configs.Layout(n=n, nsys0=nsys, row_stride=1, sys_stride0=n)
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = configs.partitioned(4, 4, n) if mode == "perrow" else configs.adi(4, 4, n)
    p = dataclasses.replace(p, layout=layout, law="perrow" if mode == "perrow" else "uniform_d")
    if mode == "shift":
        p = dataclasses.replace(p, shift=np.linspace(0.0, 2.0, nsys).astype(dtype).astype(np.float64))
    a, b, c, d = [v.astype(dtype).astype(np.float64) for v in parity.host_problem(p)]
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tol = parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32
    for opts in ({}, {"batch": 50}):
        tx = torch.full_like(td, float("nan"))
        tdma.solve_partitioned(layout, coeffs, td, tx, partitions=8, **opts)
        tdma.check()
        err = parity.per_system_error(layout, tx.double().cpu().numpy(), ref)
        assert err.max() <= tol, (opts, err.max())
