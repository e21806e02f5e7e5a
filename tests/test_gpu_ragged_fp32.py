"""FP32 ragged batches: recorded into a graph beside a strided solve (blocks of
512 lanes, 1024 for the longest systems), and with a per-system shift (one
launch per length bucket, on several streams), up to 16,384 rows.  The bar is
the plain FP32 one; replays and calls repeat bit for bit."""
import numpy as np
import pytest

import oracle
from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _f32(v):
    return v.astype(np.float32).astype(np.float64)


def _ragged(nsys, nmin, nmax, seed):
    p = configs.ragged(nsys=nsys, nmin=nmin, nmax=nmax, seed=seed)
    a, b, c, d = [_f32(v) for v in parity.host_problem(p)]
    return p, a, b, c, d


@pytest.mark.parametrize("nsys,nmin,nmax", [(300, 2, 64), (200, 500, 1000), (40, 4000, 16384), (100, 30, 9000)])
def test_fp32_ragged_graph(nsys, nmin, nmax):
    import paper_2509_03933_amd as tdma
    p, a, b, c, d = _ragged(nsys, nmin, nmax, 11)
    ref = parity.oracle_solution(p, a, b, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float32)
    (td,) = parity.to_device([d], torch.float32)
    tx = torch.full_like(td, float("nan"))
    s = configs.adi(32, 16, 256)
    sa, sb, sc, sd = [_f32(v) for v in parity.host_problem(s)]
    sco = parity.device_coeffs(s, sa, sb, sc, torch.float32)
    (tsd,) = parity.to_device([sd], torch.float32)
    ty, tz = torch.full_like(tsd, float("nan")), torch.full_like(tsd, float("nan"))
    g = tdma.graph_create([dict(layout=s.layout, coeffs=sco, d=tsd, x=ty),
                           dict(layout=p.layout, coeffs=coeffs, d=td, x=tx),
                           dict(layout=s.layout, coeffs=sco, d=ty, x=tz, after=0)])
    first = None
    for _ in range(3):
        tx.fill_(float("nan"))
        g.launch()
        tdma.check()
        err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
        assert err.max() <= parity.TOL_F32, err.max()
        first = tx.clone() if first is None else first
        assert torch.equal(tx, first)
    g.destroy()


@pytest.mark.parametrize("nsys,nmin,nmax", [(50, 8, 16), (300, 8, 64), (200, 2, 200), (60, 30, 16384)])
def test_fp32_ragged_shifted(nsys, nmin, nmax):
    import paper_2509_03933_amd as tdma
    p, a, b, c, d = _ragged(nsys, nmin, nmax, 12)
    shift = _f32(np.linspace(0.0, 1.0, nsys))
    off = p.layout.offsets
    ref = np.concatenate([oracle.thomas(a[i:j], b[i:j] + s, c[i:j], d[i:j])
                          for i, j, s in zip(off[:-1], off[1:], shift)])
    coeffs = parity.device_coeffs(p, a, b, c, torch.float32)
    coeffs["shift"] = torch.from_numpy(shift).to("cuda", torch.float32)
    (td,) = parity.to_device([d], torch.float32)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    assert err.max() <= parity.TOL_F32, err.max()
    ty = torch.full_like(td, float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, ty)
    tdma.check()
    assert torch.equal(tx, ty)
