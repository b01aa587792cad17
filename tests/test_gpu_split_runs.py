"""The split pass over long queues, where each ray gets 8, 16, 32 or 64 lanes
of a wave: queues just beyond and between the lengths where that changes, of
every kind of ray, against the oracle; and the same views with the queue cut
short, so that the rest finishes in the first pass."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_parity import assert_parity, load  # noqa: E402


def views(F, B, w, h):
    S = 65536
    a = [synth.perspective_view(synth.eye_above_floor(F, B, 33.5, 10.5), 12, 1, w, h),
         synth.perspective_view((-30.0, 140.0, 120.0), 95, -9, w, h)]
    k = synth.shadow_view(20, 30, 16, 20.0, 250.0)
    k["width"], k["height"] = w, h
    a.append(k)
    # rays along cell lines and through corners
    o = synth.ortho_view((0, 0, 200 * S), (S // 2, 0, 0), (0, 0, -S // 2), (1, 1, -0.02), w, h)
    a.append(o)
    return a


# four views of w x h rays each, nearly all of them queued after one step
@pytest.mark.parametrize("w,h", [(17, 16), (32, 33), (64, 33), (90, 47), (160, 120)])
@pytest.mark.parametrize("queue", [1 << 17, 1500])
def test_long_queues(w, h, queue):
    F, B, T = synth.make_map(250, 310, 77, dual=0.3, period=64)
    with tc.Context(0) as ctx:
        load(ctx, F, B, T)
        ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, 0)
        ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, 1)
        ctx.tc_set_option(tc.TC_OPT_SPLIT_QUEUE, queue)
        vs = views(F, B, w, h)
        print(w, h, queue, flush=True)
        wo, do = oracle.render(F, B, T, vs)
        for inline in (0, 1):
            ctx.tc_set_option(tc.TC_OPT_INLINE_TABLES, inline)
            out = tc.render(ctx, vs)
            torch.cuda.synchronize()
            assert_parity(*tc.split_hits(out), wo, do, "%dx%d queue %d" % (w, h, queue))
        assert np.count_nonzero(wo != oracle.MISS) > wo.size // 4
