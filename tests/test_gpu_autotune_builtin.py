"""The fused autotuner times the built-in rule's own shape, whatever kernel and
partition form it takes, so that a tuned solve is not slower than an untuned
one; the cached choice (uneven partitions of kernel 7 and 5 among them) keeps
parity."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _shifted(nx, ny, nz):
    p = configs.adi(nx, ny, nz)
    return dataclasses.replace(p, shift=np.linspace(0.0, 2.0, nx * ny))


# the built-in rule's (kernel, M, P) of each problem
CASES = {
    "shifted_640": (lambda: _shifted(96, 56, 640), (7, 20, 32)),
    "shifted_1000": (lambda: _shifted(4096, 2, 1000), (7, 32, 32)),
    "perrow_768": (lambda: configs.partitioned(64, 40, 768), (5, 24, 32)),
    "perrow_1000": (lambda: configs.partitioned(64, 40, 1000), (5, 32, 32)),
    "perrow_x_12": (lambda: configs.plain(nsys=60000, n=12), (0, 8, 2)),
    "shared_small": (lambda: configs.adi(16, 8, 250), (0, 16, 16)),
    "shared_short": (lambda: configs.adi(64, 64, 4), (0, 16, 1)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_builtin_shape_is_a_candidate(name):
    import paper_2509_03933_amd as tdma
    make, want = CASES[name]
    p = make()
    a, b, c, d = parity.host_problem(p)
    coeffs = parity.device_coeffs(p, a, b, c, torch.float64)
    (td,) = parity.to_device([d], torch.float64)
    tx = torch.empty_like(td)
    rec = tdma.autotune(p.layout, coeffs, td, tx, what=0)
    shapes = {(k["kernel"], k["M"], k["P"]) for k in rec["candidates"]}
    assert want in shapes, sorted(shapes)
    own = min(k["ms"] for k in rec["candidates"] if (k["kernel"], k["M"], k["P"]) == want)
    assert rec["best"]["ms"] <= own
    tx.fill_(float("nan"))
    tdma.solve_batched(p.layout, coeffs, td, tx)      # the cached shape
    tdma.check()
    ref = parity.oracle_solution(p, a, b, c, d)
    assert parity.per_system_error(p.layout, tx.cpu().numpy(), ref).max() <= parity.TOL_F64
