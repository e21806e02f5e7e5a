"""One-batch staged solves (tdma_solve_partitioned) share one workspace per
device: calls issued on several streams at once must each give what they give
alone, bit for bit, and a call recorded into a graph must replay to it."""
import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _inputs(p):
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    return parity.oracle_solution(p, a, b, c, d), coeffs, td


def test_one_batch_calls_on_several_streams():
    import paper_2509_03933_amd as tdma
    # sizes apart, so that one call's states lie where another keeps its reduced rows
    probs = [configs.partitioned(64, 32, 1024), configs.adi(48, 40, 900),
             configs.partitioned(40, 24, 300), configs.adi(100, 30, 640)]
    ins, alone = [], []
    for p in probs:
        ref, coeffs, td = _inputs(p)
        tx = torch.full_like(td, float("nan"))
        tdma.solve_partitioned(p.layout, coeffs, td, tx)
        tdma.check()
        assert parity.per_system_error(p.layout, tx.cpu().numpy(), ref).max() <= parity.TOL_F64
        ins.append((p.layout, coeffs, td))
        alone.append(tx)
    streams = [torch.cuda.Stream() for _ in probs]
    for _ in range(20):
        outs = [torch.full_like(td, float("nan")) for _, _, td in ins]
        torch.cuda.synchronize()
        for (lay, coeffs, td), tx, s in zip(ins, outs, streams):
            tdma.solve_partitioned(lay, coeffs, td, tx, stream=s)
        torch.cuda.synchronize()
        for k, (tx, want) in enumerate(zip(outs, alone)):
            assert torch.equal(tx, want), k
    tdma.check()


def test_one_batch_call_in_a_graph():
    import paper_2509_03933_amd as tdma
    p = configs.partitioned(40, 24, 300)
    ref, coeffs, td = _inputs(p)
    tx = torch.empty_like(td)
    tdma.solve_partitioned(p.layout, coeffs, td, tx)      # sizes the workspace
    torch.cuda.synchronize()
    want = tx.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        tdma.solve_partitioned(p.layout, coeffs, td, tx)
    other = configs.adi(30, 20, 200)
    _, co2, td2 = _inputs(other)
    for _ in range(4):
        tx.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(tx, want)
        tdma.solve_partitioned(other.layout, co2, td2, torch.empty_like(td2))
        torch.cuda.synchronize()
    assert parity.per_system_error(p.layout, tx.cpu().numpy(), ref).max() <= parity.TOL_F64
