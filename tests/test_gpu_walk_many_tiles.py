"""The walking kernels' built-in plans on batches of several tiles per
workgroup, with a last tile of five systems: the step from one tile to the next
on uneven partitions (kernels 7 and 5) and full ones, out of place and in
place.  Sampled systems are compared with the oracle at the parity bar, every
system with the generic kernel's solution at twice the bar (each lies within
the bar of the exact one).  And the FFT-Poisson operator, whose low modes
are ill-conditioned, on lengths that kernel 7 takes, full and uneven."""
import dataclasses

import numpy as np
import pytest

import oracle
from tests import parity
from workloads import configs, device

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (kind, dtype, n, systems per tile, tiles): at least three per resident workgroup
CASES = [("shift", "f64", 301, 32, 1600), ("shift", "f64", 512, 32, 1600), ("shift", "f64", 700, 32, 800),
         ("shift", "f64", 1000, 32, 800), ("shift", "f64", 1100, 16, 1600),
         ("perrow", "f64", 301, 32, 800), ("perrow", "f64", 512, 32, 800), ("perrow", "f64", 1000, 16, 800),
         ("perrow", "f64", 1500, 8, 800),
         ("perrow", "f32", 301, 32, 1600), ("perrow", "f32", 800, 32, 800), ("perrow", "f32", 896, 32, 800)]


@pytest.mark.parametrize("kind,dt,n,S,tiles", CASES)
def test_many_tiles(kind, dt, n, S, tiles):
    import paper_2509_03933_amd as tdma
    nsys = S * tiles + 5
    if kind == "perrow":
        p = configs.partitioned(nsys, 1, n)
    else:
        p = dataclasses.replace(configs.adi(nsys, 1, n), law="uniform_d", shift=np.linspace(0.0, 3.0, nsys))
    td, coeffs = device.device_inputs(p)
    tol = parity.TOL_F64
    if dt == "f32":
        td = td.float()
        coeffs = {k: v.float() if torch.is_tensor(v) else v for k, v in coeffs.items()}
        tol = parity.TOL_F32
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    ty = torch.full_like(td, float("nan"))
    tdma.solve_batched_tiled(p.layout, coeffs, td, ty, M=16, S=8 if dt == "f32" else 4, P=-(-n // 16))
    tdma.check()
    scale = ty.view(n, nsys).abs().amax(0).clamp_min(1e-300)
    diff = ((tx - ty).view(n, nsys).abs().amax(0) / scale).max().item()
    assert diff <= 2 * tol, diff
    systems = sorted({0, 1, S - 1, S, nsys - 1, nsys - 5, nsys - 6, *range(17, nsys, nsys // 24)})
    col = lambda t: t.view(n, nsys)[:, systems].double().cpu().numpy()
    D, X = col(td), col(tx)
    if kind == "perrow":
        A, B, C = (col(coeffs[k]) for k in "abc")
    else:
        tab = [coeffs[k].double().cpu().numpy() for k in "abc"]
        sh = coeffs["shift"].double().cpu().numpy()
    for i, s in enumerate(systems):
        a, b, c = (A[:, i], B[:, i], C[:, i]) if kind == "perrow" else (tab[0], tab[1] + sh[s], tab[2])
        ref = oracle.thomas(a, b, c, D[:, i])
        assert np.max(np.abs(X[:, i] - ref)) / np.max(np.abs(ref)) <= tol, s
    tdma.solve_batched(p.layout, coeffs, td, td)      # in place
    assert torch.equal(td, tx)


@pytest.mark.parametrize("nx,ny,n", [(128, 96, 300), (128, 64, 512), (96, 64, 640), (96, 64, 1000), (64, 64, 1024),
                                     (80, 64, 2000)])
def test_poisson_modes(nx, ny, n):
    import paper_2509_03933_amd as tdma
    p = configs.poisson(nx, ny, n)
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    x = tx.cpu().numpy()
    get = lambda q, s: x[q.layout.sys_rows(s)]
    # mode (0, 0) carries a placeholder shift in the bulk call: left out
    parity.mode_table(f"default plan {nx}x{ny}x{n}", parity.poisson_mode_rows(p, get), parity.TOL_F64)
    for s in range(11, p.layout.nsys, p.layout.nsys // 40):
        sa, sb, sc, sd = configs.system_inputs(p, s)
        ok, *err = parity.conditioned_error(get(p, s), sa, sb, sc, sd, parity.TOL_F64)
        assert ok, (s, err)
