"""Loading a map whose check is shared between threads (2^22 cells and more)
and maps with padded rows: the first bad cell in row order is the one
reported, a refused map leaves the loaded one in place, and the columns read
back are those given."""
import ctypes

import numpy as np
import pytest

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def planes(W, H):
    rng = np.random.default_rng(W + H)
    F = rng.integers(0, 200, (H, W)).astype(np.uint8)
    two = rng.random((H, W)) < 0.3
    B = np.where(two, F + 1 + rng.integers(0, 20, (H, W)), 0).astype(np.uint8)
    T = np.where(two, B + rng.integers(0, 30, (H, W)), 0).astype(np.uint8)
    return F, B, T


@pytest.mark.parametrize("bad", [[(0, 0)], [(2046, 2099)], [(5, 1700), (3, 1701)],
                                 [(2046, 261), (0, 262)], [(9, 2000), (1, 525), (7, 1050)]])
def test_first_bad_cell(bad):
    W, H = 2047, 2100
    F, B, T = planes(W, H)
    with tc.Context(0) as ctx:
        ctx.tc_load_columns(F[:9, :5], B[:9, :5], T[:9, :5])
        b2, t2 = B.copy(), T.copy()
        for x, y in bad:
            b2[y, x], t2[y, x] = 0, 1
        first = min(bad, key=lambda c: (c[1], c[0]))
        with pytest.raises(tc.TCError, match=r"\(%d,%d\)" % first):
            ctx.tc_load_columns(F, b2, t2)
        ctx.W, ctx.H = 5, 9
        for got, want in zip(ctx.tc_read_columns(0, 0, 5, 9), (F, B, T)):
            assert np.array_equal(got, want[:9, :5])
        ctx.tc_load_columns(F, B, T)
        for got, want in zip(ctx.tc_read_columns(0, 0, W, H), (F, B, T)):
            assert np.array_equal(got, want)


@pytest.mark.parametrize("W,stride", [(70, 70), (70, 71), (64, 256)])
def test_row_stride(W, stride):
    H = 33
    F, B, T = planes(stride, H)
    with tc.Context(0) as ctx:
        st = tc.load_library().tc_load_columns(ctx.handle, W, H, F.ctypes.data, B.ctypes.data,
                                               T.ctypes.data, stride, ctypes.c_void_p(0))
        assert st == tc.TC_OK
        for got, want in zip(ctx.tc_read_columns(0, 0, W, H), (F, B, T)):
            assert np.array_equal(got, want[:, :W])
