"""Host checks of the built-in tile rules (no GPU): the shape that the library's
planner chooses, asked through its internal symbol."""
import ctypes

import pytest

import paper_2509_03933_amd as tdma


class _Shape(ctypes.Structure):
    _fields_ = [("M", ctypes.c_int), ("S_log2", ctypes.c_int), ("P", ctypes.c_int), ("contig", ctypes.c_bool),
                ("kernel", ctypes.c_int), ("pdd", ctypes.c_bool)]


def _builtin(kind, dt, axis, n, nsys, run=None):
    """(kernel, M, P, systems per tile) for nsys systems of n rows: contiguous
    (x), adjacent systems (z) or planes of `run` adjacent systems (y)."""
    fn = tdma.lib()["_ZN4tdma13builtin_shapeEPK11tdma_layoutPK11tdma_coeffsiPNS_9TileShapeE"]
    fn.restype = ctypes.c_bool
    if axis == "x":
        L = tdma._Layout(n, nsys, 1, 1, n, 0)
    elif axis == "z":
        L = tdma._Layout(n, nsys, 1, max(nsys, 2), 1, 0)
    else:
        L = tdma._Layout(n, run, nsys // run, run, 1, n * run)
    C = tdma._Coeffs(tdma.COEF_LIKE_D if kind == "perrow" else tdma.COEF_SHARED, 1, 1, 1,
                     1 if kind == "shift" else None)
    sh = _Shape()
    assert fn(ctypes.byref(L), ctypes.byref(C), tdma.F64 if dt == "f64" else tdma.F32, ctypes.byref(sh))
    return sh.kernel, sh.M, sh.P, 1 << sh.S_log2


@pytest.mark.parametrize("kind", ["shared", "perrow"])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("lg", [21, 23, 26])
def test_short_contiguous_lines_fill_a_wavefront(kind, dt, lg):
    for n in range(2, 33):
        kernel, M, P, S = _builtin(kind, dt, "x", n, (1 << lg) // n)
        assert P * S >= 60, (n, kernel, M, P, S)
