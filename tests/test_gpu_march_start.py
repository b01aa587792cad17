"""The sampled march from the packet's common start, where the number of
samples skipped is small, all or none: few and many samples, near and far
limits, groups that do not divide the count, eyes above, below, beside and
far from the map.  Bit for bit the oracle's march."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_march import assert_same, gpu_march, load, set_march  # noqa: E402


def views(W, H):
    far = 30000.0
    return [synth.perspective_view(e, yaw, pitch, w, h) for e, yaw, pitch, w, h in [
        ((W / 2, H / 2, 300.0), 20, -35, 37, 21),
        ((W / 2 + 0.5, -40.0, 90.0), 0, -12, 41, 9),
        ((W / 2, H / 2, -50.0), 45, 40, 12, 12),          # below the ground
        ((-far, H / 2, 2000.0), 90, -3.8, 33, 17),        # far beside, looking in
        ((W + 5.0, H / 2, 40.0), 90, 0, 9, 9),            # looking away
        ((W / 2, H / 2, 9000.0), 0, -90, 16, 16),
        ((3.25, 3.75, 260.0), 10, 5, 10, 8),              # rising above everything
    ]]


@pytest.mark.parametrize("far,steps,bisect", [(600, 128, 4), (1, 1, 0), (50, 3, 2), (40000, 5, 1),
                                              (1 << 20, 4096, 3), (600, 4, 4), (33000, 30001, 4)])
def test_start(far, steps, bisect):
    F, B, T = synth.make_map(157, 83, 11, dual=0.3, period=16)
    with tc.Context(0) as ctx:
        load(ctx, F, B, T)
        set_march(ctx, far, steps, bisect)
        vs = views(157, 83)
        print(far, steps, bisect, flush=True)
        wo, do = oracle.march(F, B, T, vs, far=far, steps=steps, bisect=bisect)[:2]
        wg, dg = gpu_march(ctx, vs)
        assert_same(wg, dg, wo, do, "far %d steps %d" % (far, steps))
