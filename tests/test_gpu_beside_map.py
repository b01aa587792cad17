"""Rays over cells beside the map, whose index the kernels don't clamp: maps
of one cell, of a tile and around it, and one long row of tiles; eyes and rays
beside, before, behind and far from the map, along its edges and across its
corners.  Every mode against the oracle."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_march import assert_same, gpu_march, load, set_march  # noqa: E402
from test_gpu_skim import S, ortho  # noqa: E402


def views(W, H):
    k = 1 << 20
    out = [synth.perspective_view(e, yaw, pitch, 21, 13) for e, yaw, pitch in [
        ((-3.5, -2.25, 60.0), 45, -20), ((W + 2.0, H + 9.0, 90.0), 225, -30),
        ((W / 2, -30000.0, 900.0), 0, -1.7), ((32000.0, H / 2, 90.0), 270, 0),
        ((-0.25, H / 2, 40.0), 0, -5), ((W / 2, H / 2, 300.0), 10, -88)]]
    for x0, y0, d in [(-S, -S, (0, k, 0)), (W * S - S, -5 * S, (0, k, -k // 64)),
                      (-9 * S, H * S - S, (k, 0, 0)), (W * S + 9 * S, -S, (-k, 1, -k // 64)),
                      (-20 * S, -20 * S, (k, k, -k // 99)), (-31000 * S, -7 * S, (k, k // 4000, 0))]:
        out.append(ortho((x0, y0, 30 * S), (S // 8, 0, 0), (0, S // 8, 0), d, 9, 9))
    return out


@pytest.mark.parametrize("W,H", [(1, 1), (7, 9), (8, 8), (9, 64), (3, 4097), (4096, 5)])
def test_beside(W, H):
    F, B, T = synth.make_map(W, H, 3, dual=0.3, period=16)
    vs = views(W, H)
    with tc.Context(0) as ctx:
        load(ctx, F, B, T)
        wo, do = oracle.render(F, B, T, vs)[:2]
        ctx.tc_set_option(tc.TC_OPT_VOXEL_SHAPE, 2 | 1 << 8)
        for mode in (0, 4, 5):
            for passes in (0, 6):
                print(W, H, mode, passes, flush=True)
                ctx.tc_set_option(tc.TC_OPT_RENDER_MODE, mode)
                ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, passes)
                wg, dg = gpu_march(ctx, vs)
                assert np.array_equal(wg, wo)
                assert np.allclose(dg, do, rtol=1e-6, atol=0)
        for far, steps in ((600, 128), (40000, 37)):
            set_march(ctx, far, steps, 4)
            wm, dm = oracle.march(F, B, T, vs, far=far, steps=steps, bisect=4)[:2]
            wg, dg = gpu_march(ctx, vs)
            assert_same(wg, dg, wm, dm, "%dx%d far %d" % (W, H, far))
