"""Edits by tiles: cells, pyramid, masks and windows after lists at the edges
of what one launch takes -- rectangles that share a tile without meeting,
that end on tile edges, hang over the map, overlap in every order, more edits
than a ballot holds, and the longest list of the tile path and the shortest
beyond it -- on maps whose upper levels fit one block or do not.  Everything
must equal a fresh load of the oracle's edited map."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def levels(ctx):
    n = ctx.tc_pyramid_info()
    out = [("columns", ctx.tc_read_columns(0, 0, ctx.W, ctx.H))]
    out += [("level %d" % k, ctx.tc_read_pyramid(k)) for k in range(1, n + 1)]
    out += [("masks %d" % k, ctx.tc_read_occupancy(k)) for k in range(1, n + 1)]
    out += [("windows %d" % k, ctx.tc_read_window(k)) for k in range(n + 1)]
    return out


def crater(x, y, s, d):
    return dict(kind=2, x0=x, y0=y, w=s, h=s, depth=d)


def lists(W, H):
    rng = np.random.default_rng(W * 31 + H)
    mix = (synth.crater_list(5, W, H, 40, size=(1, min(40, W, H)), depth=(0, 255)) +
           synth.random_set_patches(6, W, H, 40, max_size=min(19, W, H)))
    yield "shared tile", [crater(0, 0, 3, 200), crater(4, 4, 3, 200), crater(5, 0, 2, 90),
                          crater(1, 6, 2, 255)]
    yield "tile edges", [crater(8, 8, 8, 60), crater(0, 8, 8, 70), crater(7, 15, 2, 80),
                         crater(W - 4, H - 4, 9, 99), crater(-5, -5, 9, 99)]
    yield "mixed", [mix[i] for i in rng.permutation(len(mix))]
    yield "one spot", [crater(W // 2 - k % 5, H // 2 - k % 3, 1 + k % 17, 9) for k in range(130)]
    for n in (512, 513):
        yield "%d edits" % n, synth.crater_list(n, W, H, n, size=(1, 9), depth=(1, 40))
    yield "large", [crater(W // 2 - 150, H // 2 - 150, 300, 77), crater(W // 2, H // 2, 5, 200)]


@pytest.mark.parametrize("W,H", [(1, 1), (5, 3), (8, 8), (9, 17), (70, 64), (255, 257), (600, 530),
                                 (2048, 1030), (37, 4100)])
def test_edit_tiles(W, H):
    F, B, T = synth.make_map(W, H, 900 + W, dual=0.3, period=8)
    with tc.Context(0) as ctx, tc.Context(0) as fresh:
        for name, edits in lists(W, H):
            print(W, H, name, flush=True)
            ctx.tc_load_columns(F, B, T)
            ctx.tc_apply_edit(edits)
            fresh.tc_load_columns(*oracle.apply_edits(F, B, T, edits))
            for (what, got), (_, want) in zip(levels(ctx), levels(fresh)):
                assert np.array_equal(got, want), (name, what)
