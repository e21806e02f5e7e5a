"""GPU parity of the small-batch plan (tdma_solve_batched on batches below the
walking kernels' sizes) against the oracle: one system, a few, counts and
lengths around the tiles' edges, and both sides of the size rule.  Tolerances
are the parity bars (FP64 1e-12, FP32 1e-5 against the oracle on the rounded
inputs): these operators are diagonally dominant, so their systems' errors are
a few hundred eps at most."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(kind, axis, n, n0, n1):
    if kind == "perrow":
        p = configs.partitioned(n0, n1, n)
    else:
        p = configs.adi(n0, n1, n)
        if kind == "shift":
            p = dataclasses.replace(p, shift=np.linspace(0.0, 3.0, n0 * n1))
    if axis == "x":
        lay = configs.Layout(n=n, nsys0=n0, nsys1=n1, row_stride=1, sys_stride0=n, sys_stride1=n * n0)
        p = dataclasses.replace(p, layout=lay)
    return p


@pytest.mark.parametrize("kind,axis", [("shared", "z"), ("shift", "z"), ("perrow", "z"), ("shared", "x")])
@pytest.mark.parametrize("n,n0,n1", [
    (2, 1, 1), (3, 5, 1), (15, 1, 1), (16, 3, 1), (17, 16, 1), (129, 17, 3), (1000, 1, 1), (1024, 9, 1),
    (2048, 3, 1),                        # the walking kernels' longest lines
    (520, 63, 32), (1040, 63, 24),       # just below 2^20 and 3 * 2^19 unknowns
    (1024, 64, 24), (1024, 64, 48),      # at the two lines of the rule
])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_small_batches(kind, axis, n, n0, n1, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = _problem(kind, axis, n, n0, n1)
    a, b, c, d = parity.host_problem(p)
    if dtype == np.float32:
        a, b, c, d = [v.astype(np.float32).astype(np.float64) for v in (a, b, c, d)]
        if p.shift is not None:
            p = dataclasses.replace(p, shift=p.shift.astype(np.float32).astype(np.float64))
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    tol = parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32
    assert err.max() <= tol, err.max()
    # in place: a block reads its tile whole before it writes any of it
    tdma.solve_batched(p.layout, coeffs, td, td)
    assert torch.equal(td, tx)


@pytest.mark.parametrize("kind,n,nsys", [
    # contiguous per-row lines: 8 rows per lane (up to 2,048 rows), 16 beyond;
    # lengths whose partitions fill a wavefront, leave lanes idle, or need LDS PCR
    ("perrow", 16, 40000), ("perrow", 63, 12000), ("perrow", 400, 3001), ("perrow", 720, 1501),
    ("perrow", 1537, 700), ("perrow", 2048, 520), ("perrow", 2049, 520), ("perrow", 8192, 131),
    # contiguous shared lines: tiles of 8, 16 or 32 systems, ties between row
    # counts, past the streaming kernel's lengths
    ("shared", 48, 33001), ("shared", 96, 17003), ("shared", 200, 8501), ("shared", 256, 6401),
    ("shared", 513, 3301), ("shared", 1000, 1603), ("shared", 1537, 1100), ("shared", 2049, 803),
    ("shared", 4096, 401),
])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_contiguous_line_shapes(kind, n, nsys, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = _problem(kind, "x", n, nsys, 1)
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
