"""PDD solves of more than 64 partitions, contiguous and strided, every
coefficient mode, against the oracle's PDD at the parity bar (test_gpu_pdd's
comparison)."""
import dataclasses

import numpy as np
import pytest

from tests import parity
from tests.test_gpu_pdd import _check, _solve
from workloads import configs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["shared", "shift", "perrow"])
@pytest.mark.parametrize("axis", ["x", "z"])
@pytest.mark.parametrize("m,n", [(4, 259), (4, 512), (8, 1000), (16, 2100)])
def test_many_partitions(kind, axis, m, n):
    nsys = 19
    layout = configs.Layout(n=n, nsys0=nsys, row_stride=1, sys_stride0=n) if axis == "x" else \
        configs.Layout(n=n, nsys0=nsys, row_stride=nsys, sys_stride0=1)
    p = configs.partitioned(4, 4, n) if kind == "perrow" else configs.adi(4, 4, n)
    p = dataclasses.replace(p, layout=layout, law="perrow" if kind == "perrow" else "uniform_d")
    if kind == "shift":
        p = dataclasses.replace(p, shift=np.linspace(0.5, 2.0, nsys))
    _check(p, m, _solve(p, m), parity.TOL_F64)
