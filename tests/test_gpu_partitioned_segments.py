"""GPU parity of the staged solve where Stage C's segments begin and end:
partitions with no interior row, one, a whole segment of 16, one row more or
fewer, several; every coefficient mode, in place, and one batch (the caller's
stream alone) against several.  Tolerances are the parity bars."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _problem(mode, n):
    if mode.startswith("perrow"):
        p = configs.partitioned(37, 9, n)
    else:
        p = configs.adi(37, 9, n)
    if mode.endswith("shift"):
        p = dataclasses.replace(p, shift=np.linspace(0.0, 2.0, 37 * 9))
    return p


@pytest.mark.parametrize("mode", ["perrow", "perrow_shift", "shared", "shared_shift"])
@pytest.mark.parametrize("n,P", [(2, 1), (3, 1), (17, 1), (18, 1), (19, 1), (34, 1), (35, 1), (50, 1),
                                 (56, 3), (300, 8)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_segment_edges(mode, n, P, dtype):
    import paper_2509_03933_amd as tdma
    tt = torch.float64 if dtype == np.float64 else torch.float32
    p = _problem(mode, n)
    a, b, c, d = parity.host_problem(p)
    if dtype == np.float32:
        a, b, c, d = [v.astype(np.float32).astype(np.float64) for v in (a, b, c, d)]
        if p.shift is not None:
            p = dataclasses.replace(p, shift=p.shift.astype(np.float32).astype(np.float64))
    # the oracle adds a shift to shared tables only: fold it into per-row b
    bo = b
    if mode == "perrow_shift":
        bo = (b.reshape(n, -1) + p.shift[None, :]).reshape(-1)
    ref = parity.oracle_solution(p, a, bo, c, d)
    coeffs = parity.device_coeffs(p, a, b, c, tt)
    (td,) = parity.to_device([d], tt)
    tx = torch.full_like(td, float("nan"))
    tdma.solve_partitioned(p.layout, coeffs, td, tx, partitions=P)          # one batch
    tdma.check()
    err = parity.per_system_error(p.layout, tx.double().cpu().numpy(), ref)
    assert err.max() <= (parity.TOL_F64 if dtype == np.float64 else parity.TOL_F32), err.max()
    ty = td.clone()
    tdma.solve_partitioned(p.layout, coeffs, ty, ty, partitions=P, batch=100)   # in place, four batches
    assert torch.equal(tx, ty)
