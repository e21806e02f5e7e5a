"""GPU parity of the generic kernel above 64 partitions, whose 2P interface
rows are solved in two levels (64 groups of ceil(2P / 64) rows per system):
groups that the rows fill exactly, partly, and past the last row; one to eight
systems per block, fewer systems than a block holds; contiguous and strided
rows, per-row and shared coefficients.  Tolerances are the parity bars."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind,axis", [("perrow", "x"), ("perrow", "z"), ("shared", "x"), ("shared", "z")])
@pytest.mark.parametrize("M,S,P", [(4, 8, 65), (4, 8, 96), (8, 8, 97), (8, 8, 128), (8, 4, 129), (8, 1, 375),
                                   (16, 1, 512), (8, 1, 1000), (4, 1, 1024)])
@pytest.mark.parametrize("short", [0, 1])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_two_level(kind, axis, M, S, P, short, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    n, n0, n1 = M * P - short * (2 * M + 3), 11, 3
    p = configs.partitioned(n0, n1, n) if kind == "perrow" else configs.adi(n0, n1, n)
    if axis == "x":
        lay = configs.Layout(n=n, nsys0=n0, nsys1=n1, row_stride=1, sys_stride0=n, sys_stride1=n * n0)
        p = dataclasses.replace(p, layout=lay)
    a, b, c, d = parity.host_problem(p)
    if dtype == np.float32:
        a, b, c, d = [v.astype(np.float32).astype(np.float64) for v in (a, b, c, d)]
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched_tiled(p.layout, coeffs, td, tx, M=M, S=S, P=P, kernel=0)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    assert err.max() <= (parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32), err.max()
