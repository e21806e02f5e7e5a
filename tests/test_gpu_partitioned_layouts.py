"""GPU parity of the staged solve on layouts whose consecutive systems are not
adjacent elements (contiguous rows, a system stride of two, short runs of
systems) and on short partitions, where Stage A keeps every row's factors, and
just past those limits, where it keeps states; in place and over several
batches bit for bit.  Tolerances are the parity bars."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

Layout = configs.Layout


def _runs(n, run, planes):
    """`planes` planes of `run` adjacent systems."""
    return Layout(n=n, nsys0=run, nsys1=planes, row_stride=run, sys_stride0=1, sys_stride1=n * run)


LAYOUTS = {
    "contiguous": lambda n: Layout(n=n, nsys0=300, row_stride=1, sys_stride0=n),
    "contiguous_many": lambda n: Layout(n=n, nsys0=2050, row_stride=1, sys_stride0=n),
    "stride2": lambda n: Layout(n=n, nsys0=1030, nsys1=2, row_stride=2060, sys_stride0=2, sys_stride1=2060 * n),
    "run1": lambda n: Layout(n=n, nsys0=1, nsys1=300, row_stride=300, sys_stride0=7, sys_stride1=1),
    "run2": lambda n: _runs(n, 2, 150),
    "run2_many": lambda n: _runs(n, 2, 1030),
    "run7": lambda n: _runs(n, 7, 43),
    "run8": lambda n: _runs(n, 8, 38),
    "run15": lambda n: _runs(n, 15, 20),
    "run16": lambda n: _runs(n, 16, 19),
    "single": lambda n: Layout(n=n, nsys0=1, row_stride=3),
}


def _problem(mode, layout):
    p = configs.partitioned(4, 4, layout.n) if mode.startswith("perrow") else configs.adi(4, 4, layout.n)
    law = "perrow" if mode.startswith("perrow") else "uniform_d"
    p = dataclasses.replace(p, layout=layout, law=law)
    if mode.endswith("shift"):
        p = dataclasses.replace(p, shift=np.linspace(0.0, 2.0, layout.nsys))
    return p


@pytest.mark.parametrize("mode", ["perrow", "perrow_shift", "shared", "shared_shift"])
@pytest.mark.parametrize("name", sorted(LAYOUTS))
@pytest.mark.parametrize("n,P", [(23, 8), (72, 8), (79, 8), (80, 8), (131, 3), (300, 8)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_layouts(mode, name, n, P, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = _problem(mode, LAYOUTS[name](n))
    a, b, c, d = parity.host_problem(p)
    if dtype == np.float32:
        a, b, c, d = [v.astype(np.float32).astype(np.float64) for v in (a, b, c, d)]
        if p.shift is not None:
            p = dataclasses.replace(p, shift=p.shift.astype(np.float32).astype(np.float64))
    # the oracle adds a shift to shared tables only: fold it into per-row b
    bo = b
    if mode == "perrow_shift":
        bo = b.copy()
        for s in range(p.layout.nsys):
            bo[p.layout.sys_rows(s)] += p.shift[s]
    ref = parity.oracle_solution(p, a, bo, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_partitioned(p.layout, coeffs, td, tx, partitions=P)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    assert err.max() <= (parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32), err.max()
    ty = td.clone()
    tdma.solve_partitioned(p.layout, coeffs, ty, ty, partitions=P, batch=100)   # in place, three batches
    rows = np.concatenate([p.layout.sys_rows(s) for s in range(p.layout.nsys)])
    at = torch.from_numpy(rows).cuda()
    assert torch.equal(tx[at], ty[at])
    rest = torch.ones(td.numel(), dtype=torch.bool, device="cuda")
    rest[at] = False
    assert torch.isnan(tx[rest]).all() and torch.equal(ty[rest], td[rest])       # nothing else written
