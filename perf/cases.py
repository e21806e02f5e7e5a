"""The work whose speed is followed: solves of the paper's systems as a flow
solver's step makes them, through the package's public entry points.

``draw`` gives more cases of the ranges that the listed ones stand for.  Sizes
of the listed cases are those of the benchmark and the tests, or odd ones
beside them.  The kinds of call:

  batched/perrow   every system its own a, b, c (the general solve), lines in
                   x (contiguous rows) or z (rows a plane apart)
  batched/shared   one operator for every line: the ADI momentum sweeps, x or z
  batched/shift    one operator plus a diagonal shift per line: FFT-Poisson lines
  ragged           a batch of independent systems of different lengths
  complex          the Poisson lines with complex data, half spectrum
  step             a whole FFT-Poisson solve (transforms and z-lines) by a plan
  refined          FP32 sweeps with FP64 refinement, of shared or shifted lines
  staged           the paper's three-stage pipelined solve, with its defaults
  pdd              the PDD approximation of an ADI sweep (partitions of 16 rows)
  sweeps           one ADI step recorded as a graph: x-, y- and z-sweep of a
                   field in turn, and a ragged batch beside them
"""
import math

import numpy as np
import torch

import paper_2509_03933_amd as tdma

DEV = "cuda"
MAX_POINTS = 1 << 30          # unknowns of the largest case


class Lines:
    """Layout of the lines of an (nx, ny, nz) field, x fastest."""

    def __init__(self, n, nsys0, nsys1, row_stride, sys_stride0, sys_stride1, offsets=None):
        self.n, self.nsys0, self.nsys1 = n, nsys0, nsys1
        self.row_stride, self.sys_stride0, self.sys_stride1 = row_stride, sys_stride0, sys_stride1
        self.offsets = offsets


def lines(axis, nx, ny, nz):
    if axis == "x":
        return Lines(nx, ny, nz, 1, nx, nx * ny)
    if axis == "y":
        return Lines(ny, nx, nz, nx, 1, nx * ny)
    return Lines(nz, nx, ny, nx * ny, 1, nx)


# ---------------------------------------------------------------------------
# the cases

def listed():
    return [
        # a handful of short systems on their own: latency
        dict(name="plain_64x256_f64", kind="perrow", axis="x", nx=256, ny=64, nz=1, dtype="f64"),
        # the ADI z-sweep of a 256^3 field, the benchmark's ordinary size
        dict(name="adi_z_256_f64", kind="shared", axis="z", nx=256, ny=256, nz=256, dtype="f64"),
        # an x-sweep in FP32 on a grid whose line length no tile divides
        dict(name="adi_x_250_f32", kind="shared", axis="x", nx=250, ny=200, nz=320, dtype="f32"),
        # general systems along z, a length between two tile sizes
        dict(name="perrow_z_1000_f64", kind="perrow", axis="z", nx=640, ny=500, nz=1000, dtype="f64"),
        # general systems along x (rows contiguous)
        dict(name="perrow_x_720_f64", kind="perrow", axis="x", nx=720, ny=400, nz=300, dtype="f64"),
        # independent systems of 32 ... 8192 rows
        dict(name="ragged_10000_f64", kind="ragged", nsys=10000, nmin=32, nmax=8192, dtype="f64"),
        # the Poisson lines of a 1024^3 field (the benchmark's headline)
        dict(name="poisson_z_1024_f64", kind="shift", axis="z", nx=1024, ny=1024, nz=1024, dtype="f64"),
        # the lines of a half spectrum with complex data, odd sizes
        dict(name="complex_z_500_f64", kind="complex", nx=500, ny=480, nz=500, dtype="f64"),
        # one whole FFT-Poisson solve of a 512^3 field
        dict(name="step_512_f64", kind="step", nx=512, ny=512, nz=512),
        # mixed precision on Poisson lines at the benchmark's tolerance
        dict(name="refined_poisson_512", kind="refined", op="shift", nx=512, ny=512, nz=512),
        # the staged solve of long per-row lines
        dict(name="staged_z_2048_f64", kind="staged", op="perrow", nx=512, ny=256, nz=2048, dtype="f64"),
        # one ADI step of a large field as a graph, ragged batch beside it
        dict(name="sweeps_768x512x1536_f64", kind="sweeps", nx=768, ny=512, nz=1536, nsys=10000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["perrow", "shared", "shift", "ragged", "complex", "step", "refined", "staged",
                       "pdd", "sweeps"])
    # single precision where a solver uses it: not for the Poisson operators,
    # whose low modes are too ill-conditioned for it
    op = rng.choice(["perrow", "shared", "shift"])
    dtype = rng.choice(["f64", "f64", "f32"])
    if kind in ("shift", "complex") or (kind == "staged" and op == "shift"):
        dtype = "f64"
    if kind == "ragged":
        nmin = _log(rng, 8, 64)
        return dict(kind=kind, nsys=_log(rng, 50, 40000), nmin=nmin, nmax=_log(rng, 4 * nmin, 8192),
                    dtype=dtype)
    if kind == "step":
        return dict(kind=kind, nx=_log(rng, 32, 640), ny=_log(rng, 32, 640), nz=_log(rng, 32, 1024))
    if kind == "sweeps":
        return dict(kind=kind, nx=_log(rng, 64, 768), ny=_log(rng, 64, 512), nz=_log(rng, 64, 1536),
                    nsys=_log(rng, 50, 10000))
    # line length, and how many lines: from a few to a field of 2^30 points
    # (per-row inputs, five arrays: 2^29)
    axis = rng.choice(["z", "z", "x"])
    top = {"complex": 1000, "staged": 4096}.get(kind, 1536)
    if kind == "shift" or (kind == "refined" and axis == "z"):
        top = 1024
    n = _log(rng, 32, top)
    if kind in ("perrow", "shared", "shift", "refined", "pdd") and rng.random() < 0.4:
        n = 32 * max(1, round(n / 32))      # grids are often of round sizes
    points = MAX_POINTS if kind in ("shared", "shift") else MAX_POINTS >> 2
    nsys = _log(rng, 16, min(points // n, 1 << 20))
    n0 = max(1, min(nsys, _log(rng, 16, 1024)))
    n1 = max(1, nsys // n0)
    if kind == "complex":
        return dict(kind=kind, nx=max(2, 2 * (n0 - 1)), ny=n1, nz=n, dtype=dtype)
    if kind in ("shift", "staged"):
        axis = "z"
    nx, ny, nz = (n, n0, n1) if axis == "x" else (n0, n1, n)
    if kind == "staged":
        return dict(kind=kind, op=op, nx=nx, ny=ny, nz=nz, dtype=dtype)
    if kind == "refined":
        op = "shift" if axis == "z" and rng.random() < 0.5 else "shared"
        return dict(kind=kind, op=op, axis=axis, nx=nx, ny=ny, nz=nz)
    return dict(kind=kind, axis=axis, nx=nx, ny=ny, nz=nz, dtype=dtype)


# ---------------------------------------------------------------------------
# inputs

def _torch_dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.float64


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(shape, lo, hi, gen, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).uniform_(lo, hi, generator=gen)


def _tanh_grid(n, stretch=2.0):
    """Cell widths and the centre distances over each cell's lower and upper
    face of a grid clustered at both walls of [0, 1]."""
    k = np.arange(n + 1)
    zf = 0.5 * (1.0 + np.tanh(stretch * (2.0 * k / n - 1.0)) / np.tanh(stretch))
    dz, zc = np.diff(zf), 0.5 * (zf[:-1] + zf[1:])
    h = np.diff(zc)
    return dz, zc, np.concatenate([[0.5 * dz[0]], h]), np.concatenate([h, [0.5 * dz[-1]]])


def _adi_tables(n, uniform):
    """1 - A of a Crank-Nicolson viscous sweep, Dirichlet walls, mean r = 0.5."""
    if uniform:
        lo = hi = np.full(n, 0.5)
    else:
        dz, _, h_lo, h_hi = _tanh_grid(n)
        lo, hi = 1.0 / (dz * h_lo), 1.0 / (dz * h_hi)
        s = 0.5 / (0.5 * (lo.mean() + hi.mean()))
        lo, hi = s * lo, s * hi
    a, b, c = -lo.copy(), 1.0 + lo + hi, -hi.copy()
    a[0] = c[-1] = 0.0
    return a, b, c


def _poisson_tables(n):
    """d2/dz2 on the stretched grid, Neumann walls."""
    dz, _, h_lo, h_hi = _tanh_grid(n)
    a, c = 1.0 / (dz * h_lo), 1.0 / (dz * h_hi)
    a[0] = c[-1] = 0.0
    return a, -(a + c), c


def _mode_shift(nx, ny, half):
    """Minus the modified wavenumbers of the unit box, kx fastest."""
    kx = np.arange(nx // 2 + 1 if half else nx)
    lx = (2.0 - 2.0 * np.cos(2.0 * np.pi * kx / nx)) * nx * nx
    ly = (2.0 - 2.0 * np.cos(2.0 * np.pi * np.arange(ny) / ny)) * ny * ny
    return -(ly[:, None] + lx[None, :]).reshape(-1)


def _bulk_shift(nx, ny, half):
    """The shifts with mode (0, 0), which is singular, given another mode's
    (its own pinned system is solved apart)."""
    s = _mode_shift(nx, ny, half)
    s[0] = s[1] if s.size > 1 else -1.0
    return s


def _dev(v, dtype):
    return torch.from_numpy(np.ascontiguousarray(v)).to(device=DEV, dtype=dtype)


def _smooth(nx, ny, nz, gen, dtype):
    """A smooth field with noise on it, (nz, ny, nx)."""
    ax = torch.arange(nx, device=DEV, dtype=torch.float64)
    ay = torch.arange(ny, device=DEV, dtype=torch.float64)
    az = torch.arange(nz, device=DEV, dtype=torch.float64)
    ph = torch.rand(3, device=DEV, dtype=torch.float64, generator=gen)
    f = _uniform((nz, ny, nx), -1e-3, 1e-3, gen, dtype)
    sx = torch.sin(2.0 * math.pi * ((ax + 0.5) / nx + ph[0])).to(dtype)
    sy = torch.sin(2.0 * math.pi * ((ay + 0.5) / ny + ph[1])).to(dtype)
    cz = torch.cos(math.pi * ((az + 0.5) / nz + ph[2])).to(dtype)
    return f.addcmul_(sy[:, None] * sx[None, :], cz[:, None, None])


def _perrow(size, gen, dtype, margin=None):
    """Diagonally dominant rows: a, c in (-1, 1), b = |a| + |c| + (1, 2) or
    + margin, d in (-1, 1).  The corner entries are left as they come: the
    solve does not read them."""
    a = _uniform(size, -1.0, 1.0, gen, dtype)
    c = _uniform(size, -1.0, 1.0, gen, dtype)
    b = _uniform(size, 1.0, 2.0, gen, dtype) if margin is None else margin.to(dtype)
    b = b + a.abs()
    b += c.abs()
    return a, b, c, _uniform(size, -1.0, 1.0, gen, dtype)


def _ragged(nsys, nmin, nmax, seed, dtype):
    # the lengths belong to the problem (one structure, many right-hand sides)
    gen = _gen(seed + 7)
    u = np.random.RandomState(nsys).uniform(math.log(nmin), math.log(nmax), nsys)
    rs = np.random.RandomState(int(seed) % (1 << 31))
    off = np.zeros(nsys + 1, dtype=np.int64)
    np.cumsum(np.rint(np.exp(u)).astype(np.int64), out=off[1:])
    margin = _dev(np.repeat(rs.uniform(0.01, 1.0, nsys), np.diff(off)), torch.float64)
    a, b, c, d = _perrow(int(off[-1]), gen, dtype, margin)
    lay = Lines(int(np.diff(off).max()), nsys, 1, 1, 0, 0, offsets=off)
    return lay, dict(mode=tdma.COEF_LIKE_D, a=a, b=b, c=c), d


def _shared(tables, dtype, shift=None):
    a, b, c = tables
    co = dict(mode=tdma.COEF_SHARED, a=_dev(a, dtype), b=_dev(b, dtype), c=_dev(c, dtype))
    if shift is not None:
        co["shift"] = _dev(shift, dtype)
    return co


def _pinned(tables, dtype):
    a, b, c = (v.copy() for v in tables)
    a[0] = c[0] = 0.0
    b[0] = 1.0
    return _shared((a, b, c), dtype)


def _field_inputs(case, seed):
    """(layout, coefficients, d) of a uniform case, tensors on the GPU."""
    gen, dt = _gen(seed), _torch_dtype(case)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    axis, op = case.get("axis", "z"), case.get("op", case["kind"])
    lay = lines(axis, nx, ny, nz)
    if op == "perrow":
        a, b, c, d = _perrow((nz, ny, nx), gen, dt)
        return lay, dict(mode=tdma.COEF_LIKE_D, a=a, b=b, c=c), d
    if op in ("shared", "pdd"):
        return lay, _shared(_adi_tables(lay.n, axis != "z"), dt), _smooth(nx, ny, nz, gen, dt)
    d = _uniform((nz, ny, nx), -1.0, 1.0, gen, dt)
    d[0, 0, 0] = 0.0
    return lay, _shared(_poisson_tables(nz), dt, _bulk_shift(nx, ny, False)), d


def _complex_inputs(case, seed):
    gen, dt = _gen(seed), _torch_dtype(case)
    h, ny, nz = case["nx"] // 2 + 1, case["ny"], case["nz"]
    d = torch.view_as_complex(_uniform((nz, ny, h, 2), -1.0, 1.0, gen, dt))
    d[0, 0, 0] = 0.0
    return lines("z", h, ny, nz), _shared(_poisson_tables(nz), dt, _bulk_shift(case["nx"], ny, True)), d


def _step_inputs(case, seed):
    """A source field without a mean (the Neumann problem has a solution only
    for one) and the plan's host tables."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    q = _uniform((nz, ny, nx), -1.0, 1.0, _gen(seed), torch.float64)
    q[0] -= q[0].mean()
    return q, _poisson_tables(nz), _mode_shift(nx, ny, True)


def prepare(case, seed):
    kind, dt = case["kind"], _torch_dtype(case)
    if kind == "ragged":
        lay, co, d = _ragged(case["nsys"], case["nmin"], case["nmax"], seed, dt)
        return dict(kind=kind, lay=lay, co=co, d=d, x=torch.empty_like(d))
    if kind == "step":
        q, (a, b, c), shift = _step_inputs(case, seed)
        plan = tdma.PoissonPlan(case["nx"], case["ny"], case["nz"], a, b, c, shift)
        return dict(kind=kind, plan=plan, q0=q, q=torch.empty_like(q), phi=torch.empty_like(q))
    if kind == "sweeps":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        f = _smooth(nx, ny, nz, _gen(seed), dt)
        u = [torch.empty_like(f) for _ in range(3)]
        rl, rc, rd = _ragged(case["nsys"], 32, 8192, seed, dt)
        rx = torch.empty_like(rd)
        items = [dict(layout=lines("x", nx, ny, nz), coeffs=_shared(_adi_tables(nx, True), dt), d=f, x=u[0]),
                 dict(layout=lines("y", nx, ny, nz), coeffs=_shared(_adi_tables(ny, True), dt), d=u[0],
                      x=u[1], after=0),
                 dict(layout=lines("z", nx, ny, nz), coeffs=_shared(_adi_tables(nz, False), dt), d=u[1],
                      x=u[2], after=1),
                 dict(layout=rl, coeffs=rc, d=rd, x=rx)]
        return dict(kind=kind, graph=tdma.graph_create(items), out=u + [rx])
    if kind == "complex":
        lay, co, d = _complex_inputs(case, seed)
    else:
        lay, co, d = _field_inputs(case, seed)
    st = dict(kind=kind, lay=lay, co=co, d=d, x=torch.empty_like(d))
    if kind in ("shift", "complex") or case.get("op") == "shift":
        st["pin_lay"] = Lines(lay.n, 1, 1, lay.row_stride, 1, 1)
        st["pin_co"] = _pinned(_poisson_tables(lay.n), dt)
    return st


def run(st):
    kind = st["kind"]
    if kind == "sweeps":
        st["graph"].launch()
        return st["out"]
    if kind == "step":
        # the transform may use q as scratch; a solver forms it anew each step
        st["q"].copy_(st["q0"])
        st["plan"].solve(st["q"], st["phi"])
        return st["phi"]
    if kind == "complex":
        def solve(lay, co):
            tdma.solve_complex(lay, co, st["d"], st["x"])
    elif kind == "refined":
        def solve(lay, co):
            tdma.solve_refined(lay, co, st["d"], st["x"], max_iters=2, tol=1e-13, criterion=1, report=False)
    elif kind == "staged":
        def solve(lay, co):
            tdma.solve_partitioned(lay, co, st["d"], st["x"])
    elif kind == "pdd":
        def solve(lay, co):
            tdma.solve_pdd(lay, co, st["d"], st["x"], 16)
    else:
        def solve(lay, co):
            tdma.solve_batched(lay, co, st["d"], st["x"])
    solve(st["lay"], st["co"])
    if "pin_lay" in st:                     # mode (0, 0), on the same arrays
        solve(st["pin_lay"], st["pin_co"])
    return st["x"]


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    kind = case["kind"]
    esz = 4 if case.get("dtype") == "f32" else 8
    if kind == "ragged":
        # mean of the log-uniform length
        n = case["nsys"] * (case["nmax"] - case["nmin"]) / math.log(case["nmax"] / case["nmin"])
        return dict(bytes=5 * esz * n, flops=9 * n)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    op = case.get("op", kind)
    if kind == "sweeps":
        r = case["nsys"] * (8192 - 32) / math.log(8192 / 32)
        return dict(bytes=3 * 16 * n + 40 * r, flops=3 * 5 * n + 9 * r)
    if kind == "step":
        # the copy of q, and the solve: two transforms and the complex lines
        return dict(bytes=4 * 8 * n, flops=n * (5 * math.log2(nx * ny) + 14))
    if kind == "complex":
        m = (nx // 2 + 1) * ny * nz
        return dict(bytes=4 * esz * m, flops=14 * m)
    if op == "perrow":
        return dict(bytes=5 * esz * n, flops=9 * n)
    sweeps = 5 if kind == "refined" else 1   # three solves and two residuals
    return dict(bytes=2 * esz * n, flops=sweeps * (9 if op == "shift" else 5) * n)


# ---------------------------------------------------------------------------
# 64-bit results, by the Thomas algorithm over all systems at once

def _thomas(a, b, c, d):
    """Rows along dim 0; a, b, c broadcast against d's systems.  d (which may
    be complex) is overwritten with x."""
    n = d.shape[0]
    cp = torch.empty_like(b)
    cp[0] = c[0] / b[0]
    d[0] /= b[0]
    for i in range(1, n):
        m = 1.0 / (b[i] - a[i] * cp[i - 1])
        cp[i] = c[i] * m
        d[i] = (d[i] - a[i] * d[i - 1]) * m
    for i in range(n - 2, -1, -1):
        d[i] -= cp[i] * d[i + 1]
    return d


def _thomas_shared(co, d):
    """Shared tables (with a shift, one per system) over d of (n, systems)."""
    a, b, c = (co[k].double() for k in "abc")
    one = (d.shape[0], 1)
    if "shift" in co:
        b = b[:, None] + co["shift"].double()[None, :]
        a, c = a.reshape(one), c.reshape(one)
        n = d.shape[0]
        cp = torch.empty_like(b)
        cp[0] = c[0] / b[0]
        d[0] /= b[0]
        for i in range(1, n):
            m = 1.0 / (b[i] - a[i] * cp[i - 1])
            cp[i] = c[i] * m
            d[i] = (d[i] - a[i] * d[i - 1]) * m
        for i in range(n - 2, -1, -1):
            d[i] -= cp[i] * d[i + 1]
        return d
    return _thomas(a.reshape(one), b.reshape(one), c.reshape(one), d)


def _rows_first(v, axis):
    """The (nz, ny, nx) field as (rows, ...) along an axis (a view)."""
    return v.movedim({"z": 0, "y": 1, "x": 2}[axis], 0)


def _exact_ragged(lay, co, d):
    lens = np.diff(lay.offsets)
    order = np.argsort(-lens, kind="stable")
    off = torch.from_numpy(lay.offsets[:-1][order].copy()).to(DEV)
    sorted_lens = lens[order]
    a, b, c = (co[k].double() for k in "abc")
    x = d.double().clone()
    cp = torch.zeros_like(x)
    count = np.searchsorted(-sorted_lens, -np.arange(1, sorted_lens[0] + 1), side="right")
    x[off] /= b[off]
    cp[off] = c[off] / b[off]
    for i in range(1, int(sorted_lens[0])):
        k = off[:count[i]] + i
        m = 1.0 / (b[k] - a[k] * cp[k - 1])
        cp[k] = c[k] * m
        x[k] = (x[k] - a[k] * x[k - 1]) * m
    # c of a system's last row is not part of it
    cp[torch.from_numpy(lay.offsets[1:] - 1).to(DEV)] = 0.0
    for i in range(int(sorted_lens[0]) - 2, -1, -1):
        k = off[:count[i + 1]] + i
        x[k] -= cp[k] * x[k + 1]
    return x


def _exact_pdd(case, co, d, m=16):
    """The approximation itself: blocks of m rows solved apart, the two
    unknowns at each block boundary from 2 x 2 systems."""
    a, b, c = (co[k].double() for k in "abc")
    n = d.shape[0]
    nb = -(-n // m)
    x = torch.empty_like(d)
    tips = []
    for p in range(nb):
        r = slice(p * m, min(n, (p + 1) * m))
        ln = r.stop - r.start
        av, bv, cv = a[r].clone(), b[r], c[r].clone()
        v = torch.zeros(ln, 1, dtype=torch.float64, device=DEV)
        w = torch.zeros_like(v)
        if p:
            v[0] = av[0]
        if p < nb - 1:
            w[-1] = cv[-1]
        av[0] = cv[-1] = 0.0
        t = [z.reshape(ln, 1) for z in (av, bv, cv)]
        tips.append((_thomas(*t, v), _thomas(*t, w), r))
        x[r] = _thomas(*t, d[r].clone())
    left = [torch.zeros_like(x[0])] * nb
    right = [torch.zeros_like(x[0])] * nb
    for p in range(nb - 1):
        wl, vf = tips[p][1][-1], tips[p + 1][0][0]
        xl, xf = x[tips[p][2].stop - 1], x[tips[p + 1][2].start]
        det = 1.0 - wl * vf
        right[p] = (xf - vf * xl) / det
        left[p + 1] = (xl - wl * xf) / det
    for p in range(nb):
        v, w, r = tips[p]
        shape = (v.shape[0],) + (1,) * (x.dim() - 1)
        x[r] = x[r] - v.reshape(shape) * left[p] - w.reshape(shape) * right[p]
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "ragged":
        lay, co, d = _ragged(case["nsys"], case["nmin"], case["nmax"], seed, _torch_dtype(case))
        return _exact_ragged(lay, co, d)
    if kind == "step":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        q, tables, shift = _step_inputs(case, seed)
        s = torch.fft.rfft2(q)
        shift[0] = shift[1] if shift.size > 1 else -1.0
        spec = s.reshape(nz, -1)
        pin = _thomas_shared(_pinned(tables, torch.float64), spec[:, :1].clone())
        _thomas_shared(_shared(tables, torch.float64, shift), spec)
        spec[:, :1] = pin
        return torch.fft.irfft2(s, s=(ny, nx))
    if kind == "sweeps":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        f = _smooth(nx, ny, nz, _gen(seed), torch.float64)
        out = []
        for axis, n in (("x", nx), ("y", ny), ("z", nz)):
            co = _shared(_adi_tables(n, axis != "z"), torch.float64)
            g = _rows_first(f, axis).clone(memory_format=torch.contiguous_format).reshape(n, -1)
            g = _thomas_shared(co, g)
            shape = [nz, ny, nx]
            k = {"z": 0, "y": 1, "x": 2}[axis]
            f = g.reshape([shape.pop(k)] + shape).movedim(0, k).contiguous()
            out.append(f)
        lay, co, d = _ragged(case["nsys"], 32, 8192, seed, torch.float64)
        return out + [_exact_ragged(lay, co, d)]
    if kind == "complex":
        lay, co, d = _complex_inputs(case, seed)
        x = d.to(torch.complex128).reshape(lay.n, -1)
        pin = _thomas_shared(_pinned_as(case, lay.n), x[:, :1].clone())
        _thomas_shared(co, x)
        x[:, :1] = pin
        return x.reshape(d.shape)
    lay, co, d = _field_inputs(case, seed)
    axis = case.get("axis", "z")
    rows = _rows_first(d.double(), axis).contiguous()
    shape = rows.shape
    if kind == "pdd":
        x = _exact_pdd(case, co, rows)
        return x.movedim(0, {"z": 0, "y": 1, "x": 2}[axis])
    if co["mode"] == tdma.COEF_LIKE_D:
        a, b, c = (_rows_first(co[k].double(), axis).contiguous() for k in "abc")
        x = _thomas(a, b, c, rows)
    else:
        g = rows.reshape(lay.n, -1)
        pin = None
        if "shift" in co:
            pin = _thomas_shared(_pinned_as(case, lay.n), g[:, :1].clone())
        x = _thomas_shared(co, g)
        if pin is not None:
            x[:, :1] = pin
        x = x.reshape(shape)
    return x.movedim(0, {"z": 0, "y": 1, "x": 2}[axis])


def _pinned_as(case, n):
    """The pinned operator as the case's type holds it."""
    return _pinned(_poisson_tables(n), _torch_dtype(case))
