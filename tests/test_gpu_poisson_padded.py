"""FFT-Poisson plans whose half spectrum has padded rows and planes (ny a power
of two from 64 to 512, at least 16 columns of modes), and grids just outside
that rule, against the oracle's step (the bound of test_gpu_poisson_fft), twice
on one plan.  The distance from the field itself is printed, not judged: it is
the rounding of the pinned mode (0, 0), whose solution is up to a thousand
times the field here, the same with and without padding to all digits printed
(33 x 64 x 70: 6.09e-11, the oracle's step 3.87e-12)."""
import numpy as np
import pytest

from oracle import poisson as op
from tests.test_gpu_poisson_fft import _apply, _case, _off_constant

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [(30, 64, 33), (33, 64, 70), (62, 64, 40), (100, 128, 48), (64, 256, 32),
                                  (40, 512, 16), (30, 64, 1024),
                                  (28, 64, 33), (62, 48, 40), (34, 32, 40), (32, 1024, 6)])
def test_padded_spectrum(grid):
    import paper_2509_03933_amd as tdma
    nx, ny, nz = grid
    a, b, c, shift, _, _ = _case(nx, ny, nz, 0)
    plan = tdma.PoissonPlan(nx, ny, nz, a, b, c, shift)
    for seed in (1, 2):
        phi = np.random.default_rng(seed).uniform(-1, 1, nx * ny * nz)
        q = _apply(phi, nx, ny, nz, 1.0 / nx, 1.0 / ny, a, b, c)
        ref = op.poisson_fft(q, nx, ny, nz, a, b, c, shift)
        tq = torch.from_numpy(q).cuda()
        tp = torch.full_like(tq, float("nan"))
        plan.solve(tq, tp)
        tdma.check()
        got = tp.cpu().numpy()
        e_gpu, e_orc = _off_constant(got, phi), _off_constant(ref, phi)
        vs = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
        print(f"{grid}: GPU vs field {e_gpu:.2e}, oracle vs field {e_orc:.2e}, GPU vs oracle {vs:.2e}", flush=True)
        assert vs <= max(20 * e_orc, 1e-12)
    plan.destroy()
