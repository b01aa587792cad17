"""The height margin of the single-precision walk: rays that pass the edges of
plateaus and slabs within a few units (2^-16 of a height) of their heights,
from origins near and far below and above, where an origin's height is exact in
single precision and where it is not.  Records are the oracle's."""
import numpy as np
import pytest

import oracle
from synth.views import VIEW_DTYPE

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_parity import assert_parity, load  # noqa: E402

S = 65536
W, H = 160, 96


def terrain():
    rng = np.random.default_rng(11)
    F = np.kron(rng.choice([0, 1, 100, 128, 200], (H // 8, W // 8)), np.ones((8, 8))).astype(np.uint8)
    two = np.kron(rng.random((H // 4, W // 4)) < 0.3, np.ones((4, 4))) > 0
    B = np.where(two, np.minimum(F.astype(int) + rng.choice([1, 40, 55], (H, W)), 255), 0)
    T = np.where(two, np.minimum(B + rng.choice([0, 3], (H, W)), 255), 0)
    F[:, -8:] = 255
    two[:, -8:] = False
    B, T = np.where(two, B, 0), np.where(two, T, 0)
    return F, B.astype(np.uint8), T.astype(np.uint8)


def rays(F, B, T, lo, hi, n=4000):
    """1x1 views whose ray crosses a line of x at most 3 units from a height of
    the column behind it, after a way of lo..hi heights."""
    rng = np.random.default_rng([3, int(lo * 16), int(hi * 16)])
    v = np.zeros(n, VIEW_DTYPE)
    v["width"] = v["height"] = 1
    for i in range(n):
        x, y = int(rng.integers(2, W)), int(rng.integers(0, H))
        s = 1 if rng.random() < 0.5 else -1
        h = int(rng.choice([F[y, x], B[y, x], T[y, x], F[y, x - 1]]))
        z = h * S + int(rng.integers(-3, 4))
        rise = int(rng.uniform(lo, hi) * S) * (1 if rng.random() < 0.5 else -1)
        dist = int(rng.uniform(0.3, 120) * S)        # along x
        dx = int(rng.integers(1 << 19, 1 << 22))
        dz = -(-rise * dx // dist) if rise < 0 else rise * dx // dist
        if abs(dz) >= 1 << 23:
            dx = max(1, dx * ((1 << 22)) // abs(dz))
            dz = rise * dx // dist
        dy = int(rng.integers(-dx, dx + 1)) // int(rng.choice([1, 7, 1000]))
        ox, oy = x * S - s * dist, y * S + int(rng.integers(0, S)) - dy * dist // dx
        oz = z - dz * dist // dx
        v[i]["o0"], v[i]["d0"] = (ox, oy, oz), (s * dx, dy, dz)
    return v


@pytest.mark.parametrize("beam", [0, 6])
@pytest.mark.parametrize("lo,hi", [(0, 0.001), (0, 2), (1, 60), (50, 300), (255, 259), (400, 900), (5000, 30000)])
def test_margin(lo, hi, beam):
    F, B, T = terrain()
    vs = rays(F, B, T, lo, hi)
    with tc.Context(0) as ctx:
        load(ctx, F, B, T)
        ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, beam)
        ctx.tc_set_option(tc.TC_OPT_VOXEL_SHAPE, 2 | 2 << 8)
        wo, do = oracle.render(F, B, T, vs)
        for mode in (0, 4, 5):
            print(lo, hi, beam, mode, flush=True)
            ctx.tc_set_option(tc.TC_OPT_RENDER_MODE, mode)
            out = tc.render(ctx, vs)
            torch.cuda.synchronize()
            assert_parity(*tc.split_hits(out), wo, do, "rise %g..%g mode %d" % (lo, hi, mode))
    assert np.count_nonzero(wo != oracle.MISS) > wo.size // 4
