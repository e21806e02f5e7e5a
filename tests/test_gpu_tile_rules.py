"""GPU parity of the built-in tile rules' corners: lines shorter than a
wavefront's worth of lanes, the lengths and batch sizes on either side of each
rule's line, last tiles with a single system; out of place and in place.
Tolerances are the parity bars."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

Layout = configs.Layout


def _layout(axis, n, nsys):
    if axis == "x":
        return Layout(n=n, nsys0=nsys, row_stride=1, sys_stride0=n)
    if axis == "z":
        return Layout(n=n, nsys0=nsys, row_stride=max(2, nsys), sys_stride0=1)
    run = 48                                  # y-lines: planes of 48 systems
    planes = (nsys + run - 1) // run
    return Layout(n=n, nsys0=run, nsys1=planes, row_stride=run, sys_stride0=1, sys_stride1=n * run)


# (kind, dtype, axis, n, systems)
SMALL = [(kind, dt, axis, n, nsys)
         for kind in ("shared", "shift", "perrow") for dt in ("f64", "f32") for axis in ("x", "z")
         for n, nsys in ((2, 1), (2, 129), (3, 40001), (8, 65), (15, 700), (16, 1000), (17, 65), (27, 130),
                         (40, 33), (48, 4097), (49, 31), (130, 5), (600, 9))]
SMALL += [(kind, dt, "z", n, nsys)
          for kind in ("shared", "shift", "perrow") for dt in ("f64", "f32")
          for n, nsys in ((2048, 17), (2049, 17), (1024, 15), (1025, 1100), (512, 2049), (40, 27001))]
CONTIG = [(kind, dt, "x", n, nsys)
          for kind in ("shared", "perrow") for dt in ("f64", "f32")
          for n, nsys in ((2, 300), (8, 257), (9, 1000), (14, 513), (20, 80001), (24, 65537), (31, 51001), (16, 98305),
                          (6, 174801), (40, 39401))]
LONG = [("shared", dt, "x", n, nsys) for dt in ("f64", "f32")
        for n, nsys in ((2000, 265), (2100, 255), (3000, 511), (3000, 513), (6000, 215), (6000, 257))]
SHIFTED = [("shift", "f64", axis, n, nsys) for axis in ("y", "z")
           for n, nsys in ((897, 3600), (1000, 3201), (1000, 5001), (1300, 2500), (1900, 1105), (2048, 1100))]
PERROW32 = [("perrow", "f32", axis, n, nsys) for axis in ("y", "z")
            for n, nsys in ((64, 1000), (128, 31), (64, 8300), (1000, 1700), (1024, 4001), (2048, 1009))]
CASES = SMALL + CONTIG + LONG + SHIFTED + PERROW32


@pytest.mark.parametrize("kind,dt,axis,n,nsys", CASES)
def test_rule_corner(kind, dt, axis, n, nsys):
    import paper_2509_03933_amd as tdma
    tt, tol = (torch.float64, parity.TOL_F64) if dt == "f64" else (torch.float32, parity.TOL_F32)
    p = configs.partitioned(4, 4, n) if kind == "perrow" else configs.adi(4, 4, max(n, 4))
    layout = _layout(axis, n, nsys)
    tables = {} if kind == "perrow" else dict(a=p.a[:n], b=p.b[:n], c=p.c[:n])
    p = dataclasses.replace(p, layout=layout, law="perrow" if kind == "perrow" else "uniform_d", **tables)
    if kind == "shift":
        p = dataclasses.replace(p, shift=np.linspace(0.0, 2.0, layout.nsys))
    a, b, c, d = parity.host_problem(p)
    if dt == "f32":
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
    assert err.max() <= tol, err.max()
    tdma.solve_batched(p.layout, coeffs, td, td)      # in place
    got = parity.gather_rows(p.layout, td.cpu().numpy())
    assert np.array_equal(got, parity.gather_rows(p.layout, tx.cpu().numpy()))
