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

@pytest.mark.parametrize("kind", ["shared", "shift", "perrow"])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("axis", ["x", "z"])
def test_small_batches_of_short_lines_share_blocks(kind, dt, axis):
    """No block of a lane or two where systems enough are there to share one."""
    for lg in (13, 16, 18, 19, 20, 21):
        for n in list(range(2, 34)) + [40, 48, 49, 64, 100]:
            nsys = (1 << lg) // n
            kernel, M, P, S = _builtin(kind, dt, axis, n, nsys)
            assert P * S >= 16, (n, nsys, kernel, M, P, S)
            if axis == "z" and kernel in (0, 1):      # one tile per block
                assert P * S >= 48 or S >= nsys, (n, nsys, kernel, M, P, S)


@pytest.mark.parametrize("dt,kind,axis,n,nsys,run,walking", [
    ("f64", "shared", "z", 40, (1 << 21) // 40, None, True),
    ("f64", "shared", "z", 40, (1 << 19) // 40, None, False),
    ("f64", "shared", "y", 2000, 1536, 256, True),
    ("f64", "shared", "y", 2000, 768, 256, False),
    ("f32", "shared", "z", 640, (1 << 21) // 640, None, True),
    ("f64", "shift", "y", 2000, 1024, 256, True),
    ("f64", "shift", "y", 2000, 256, 256, False),
    ("f64", "perrow", "y", 512, 2304, 256, True),
    ("f64", "perrow", "y", 512, 1536, 256, False),
    ("f32", "perrow", "z", 1024, 8, None, True),
    ("f64", "shared", "x", 8, 30000, None, True),
    ("f64", "shared", "x", 16, 30000, None, False)])
def test_small_rule_gives_way_to_the_walking_kernels(dt, kind, axis, n, nsys, run, walking):
    kernel, M, P, S = _builtin(kind, dt, axis, n, nsys, run)
    small = kernel == 0 or (kind == "shared" and dt == "f32" and kernel == 1)
    assert small != walking, (kernel, M, P, S)


@pytest.mark.parametrize("kind", ["shared", "shift"])
def test_lines_past_the_walking_kernels_keep_wide_tiles(kind):
    for n in (2500, 4096):
        for lg in (20.2, 20.9, 21.4):
            assert _builtin(kind, "f64", "z", n, int(2 ** lg / n))[3] > 1, (n, lg)

@pytest.mark.parametrize("n,nsys,dt,S", [(6000, 215, "f32", 1), (6000, 700, "f32", 2), (3000, 925, "f32", 4),
                                         (3000, 10000, "f64", 2), (2500, 250, "f64", 1)])
def test_few_long_contiguous_lines_take_a_block_each(n, nsys, dt, S):
    assert _builtin("shared", dt, "x", n, nsys)[3] == S


def test_contiguous_shared_lines_of_8_rows_per_lane_from_2_19():
    assert _builtin("shared", "f64", "x", 2000, 400)[1] == 8
    assert _builtin("shared", "f64", "x", 2000, 100)[1] == 4

@pytest.mark.parametrize("n,nsys,run,kernel", [
    (1000, 1 << 12, 256, 3), (1000, 1 << 13, 256, 3), (1000, 1 << 15, 256, 7), (2000, 1 << 12, 256, 3),
    (2000, 1 << 14, 256, 7), (2048, 1 << 12, 256, 3), (1300, 1 << 11, 256, 3), (1300, 1 << 12, 256, 7),
    (700, 1 << 13, 256, 7), (1024, 1 << 12, 256, 7), (1000, 1 << 13, 1 << 13, 7)])
def test_few_tiles_of_long_shifted_lines_take_kernel_3(n, nsys, run, kernel):
    """Kernel 7 needs tiles enough, or rows far apart (the last case)."""
    assert _builtin("shift", "f64", "y", n, nsys, run)[0] == kernel

@pytest.mark.parametrize("n,nsys,M,P,S", [(64, 1000, 16, 4, 16), (128, 1000, 16, 8, 16), (64, 100000, 32, 2, 128),
                                          (1024, 2000, 32, 32, 16), (1024, 5000, 32, 32, 32), (2048, 900, 32, 64, 8),
                                          (2048, 2100, 32, 64, 16)])
def test_fp32_per_row_lines_of_few_tiles(n, nsys, M, P, S):
    assert _builtin("perrow", "f32", "z", n, nsys)[1:] == (M, P, S)
