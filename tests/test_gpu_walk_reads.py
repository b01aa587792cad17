"""How many nodes and cells a walk reads where single precision decides
little: rays a unit above a plateau, shadow rays of a level light, rays along
cell lines.  Each is counted against rays of the same kind that rounding
leaves nothing open for, and every record is the oracle's.  A walk that goes
through such a stretch cell by cell reads hundreds per ray more.  Rays through
corners read no more; they are timed."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_parity import assert_parity, load  # noqa: E402
from test_gpu_shade import assert_same  # noqa: E402
from test_gpu_skim import S, ortho  # noqa: E402

K = 1 << 22
N = 600       # cells a ray runs along the plateau
LEVELS = 10   # of a 640-cell map: a walk climbs them and comes down again


@pytest.fixture()
def ctx():
    with tc.Context(0) as c:
        c.tc_set_option(tc.TC_OPT_COUNT_READS, 1)
        yield c


def counted(ctx, F, B, T, views, what):
    ctx.tc_read_counters()
    out = tc.render(ctx, views)
    torch.cuda.synchronize()
    n = ctx.tc_read_counters()
    wo, do = oracle.render(F, B, T, views)
    assert_parity(*tc.split_hits(out), wo, do, what)
    return n / wo.size


def plateau(axis):
    F = np.full((640, 640), 100, np.uint8)
    F[:, 10 + N:] = 140
    F = F if axis == 0 else np.ascontiguousarray(F.T)
    return F, np.zeros_like(F), np.zeros_like(F)


# rays 1, 20 and 40 units above the plateau, against rays 2,048 above it (a
# 32nd of a cell: within the packet beam's margin, so both kinds begin alike)
@pytest.mark.parametrize("axis,slope", [(0, 0), (0, 9), (1, 0), (1, -11)])
@pytest.mark.parametrize("mode,budget,w", [(0, 0, 40), (0, 5, 8), (0, 5, 70), (4, 0, 40), (5, 0, 40)])
def test_plateau(ctx, mode, budget, w, axis, slope):
    F, B, T = plateau(axis)
    ctx.tc_set_option(tc.TC_OPT_VOXEL_SHAPE, 4 | 2 << 8)
    ctx.tc_set_option(tc.TC_OPT_RENDER_MODE, mode)
    ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, budget)
    load(ctx, F, B, T)
    d = (K, slope * K // 100) if axis == 0 else (slope * K // 100, K)
    o = (9 * S + 3, 200 * S + 77) if axis == 0 else (200 * S + 77, 9 * S + 3)
    step = (0, S, 0) if axis == 0 else (S, 0, 0)

    def view(dz):
        return ortho(o + (100 * S + dz,), step, (0, 0, 0), d + (0,), w, 20)

    got = {}
    for dz in (2048, 1, 20, 40):
        print(mode, budget, w, axis, slope, dz, flush=True)
        got[dz] = counted(ctx, F, B, T, [view(dz)], "%d above" % dz)
    # one more climb and descent, of two reads a level each at the most
    for dz in (1, 20, 40):
        runs = 1 if budget == 0 or w > 50 else 256   # (a run of its own per cell)
        assert got[dz] <= got[2048] + 4 * LEVELS * min(runs, 64), got


# a step at x = 4 and beyond it a plateau as high as the step, or one lower
@pytest.mark.parametrize("light", [(K, 0, 0), (K, 1234567, 0), (K, -7, 5), (K, K // 3, 400)])
def test_level_light(ctx, light):
    pal = synth.default_palette()
    got = {}
    for far in (99, 100):
        F = np.full((64, 640), 100, np.uint8)
        F[:, 5:8] = 99
        F[:, 8:] = far
        Z = np.zeros_like(F)
        load(ctx, F, Z, Z)
        # straight down on the step's top, whose normal leans to the light
        v = ortho((4 * S, 0, 200 * S), (S // 64, 0, 0), (0, S // 2, 0), (0, 0, -K), 32, 48)
        hits = tc.render(ctx, [v])
        rgba = torch.empty(32 * 48, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        ctx.tc_read_counters()
        print(light, far, flush=True)
        ctx.tc_shade_views([v], hits.data_ptr(), light, pal, rgba.data_ptr())
        torch.cuda.synchronize()
        got[far] = ctx.tc_read_counters() / (32 * 48)
        assert_same(rgba.cpu().numpy().view(np.uint32), oracle.shade(F, Z, Z, [v], light, pal), str(light))
    assert got[100] <= got[99] + 4 * LEVELS, got


# every ray on a cell line, against the same rays half a cell beside it, over
# a map that is the same along the other axis: both begin in the cell where
# the beam ends, and read the same
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("mode", [0, 4, 5])
def test_cell_lines(ctx, mode, axis, sign):
    prof = synth.make_map(640, 64, 5, dual=0.2, period=64)
    F, B, T = (np.ascontiguousarray(np.repeat(p[:1], 640, 0)) for p in prof)
    if axis == 1:
        F, B, T = (np.ascontiguousarray(p.T) for p in (F, B, T))
    ctx.tc_set_option(tc.TC_OPT_VOXEL_SHAPE, 4 | 2 << 8)
    ctx.tc_set_option(tc.TC_OPT_RENDER_MODE, mode)
    ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, 0)
    load(ctx, F, B, T)
    got = {}
    for off in (S // 2, 0):
        along, across = (-40 * S if sign > 0 else 680 * S) + 5, 100 * S + off
        o = (along, across, 90 * S) if axis == 0 else (across, along, 90 * S)
        d = (sign * K, 0, -K // 30) if axis == 0 else (0, sign * K, -K // 30)
        step = (0, S // 2, 0) if axis == 0 else (S // 2, 0, 0)
        print(mode, axis, sign, off, flush=True)
        got[off] = counted(ctx, F, B, T, [ortho(o, step, (0, 0, S // 4), d, 64, 300)], "offset %d" % off)
    # (the beam's boxes of the two lie half a cell apart)
    assert abs(got[0] - got[S // 2]) <= 0.02 * got[S // 2], got


# rays that meet a corner at every crossing, against those that pass beside
# them: the exact order of two crossings costs as much again as the step, not
# several times as much (medians of the kernels' own times, in turn)
@pytest.mark.parametrize("d", [(K, K), (-K, K), (K // 3, 3 * (K // 3))])
def test_corner_time(ctx, d):
    F, B, T = synth.make_map(1024, 1024, 6, dual=0.2, period=128)
    ctx.tc_set_option(tc.TC_OPT_COUNT_READS, 0)
    ctx.tc_set_option(tc.TC_OPT_KERNEL_TIMING, 1)
    load(ctx, F, B, T)
    out = torch.empty((1000 * 1000, 2), dtype=torch.int32, device="cuda")
    ms = {0: [], 12345: []}
    for _ in range(15):
        for off in ms:
            v = ortho((off if d[0] > 0 else 1024 * S - off, 0, 260 * S), (S // 2 * (1 if d[0] > 0 else -1), 0, 0),
                      (0, S // 2, 0), d + (-K // 24,), 1000, 1000)
            ctx.tc_render_views([v], out.data_ptr())
            ms[off].append(sum(ctx.tc_read_kernel_times()))
    on, beside = (np.median(ms[k][3:]) for k in (0, 12345))
    print(d, on, beside, flush=True)
    assert on <= 2.0 * beside, (on, beside)


def rough(ctx):
    F, B, T = synth.make_map(250, 310, 78, dual=0.3, period=64)
    load(ctx, F, B, T)
    v = [synth.perspective_view(synth.eye_above_floor(F, B, 33.5, 10.5), 12, 1, 160, 120)]
    ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, 0)

    def reads(budget, boost=0):
        ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, budget)
        ctx.tc_set_option(tc.TC_OPT_PRIORITY_BOOST, boost)
        print(budget, boost, flush=True)
        return counted(ctx, F, B, T, v, "budget %d boost %d" % (budget, boost))
    return reads


# the runs of the split pass read more than the walk they take the place of,
# so a walk that reaches them shows in the count
def test_split_budget_is_the_one_set(ctx):
    reads = rough(ctx)
    never = reads(0)
    assert reads(20) > never
    assert reads(120) > never        # the default: fewer in a launch this small
    for budget in (119, 121, 1 << 20):
        assert reads(budget) == never   # no walk of this view is as long


# a wave's priority is raised within the budget, not before it begins
@pytest.mark.parametrize("queue", [1 << 17, 1500])
def test_priority_boost_leaves_the_budget(ctx, queue):
    ctx.tc_set_option(tc.TC_OPT_SPLIT_QUEUE, queue)
    reads = rough(ctx)
    never = reads(0)
    for boost in (3, 9, 1000, 1 << 20):
        assert reads(20, boost) > never
        assert reads(1 << 20, boost) == never


# steps that fall one height a cell, and rays that fall with them, 20 units
# above every edge, from so far that the margin covers it: each cell is passed
# in whole numbers, and the budget still ends
@pytest.mark.parametrize("boost", [0, 7])
def test_passed_cells_use_the_budget(ctx, boost):
    F = np.zeros((64, 640), np.uint8)
    F[:, :200] = 220 - np.arange(200)
    F[:, 205:] = 40
    Z = np.zeros_like(F)
    load(ctx, F, Z, Z)
    v = ortho((-2000 * S, 10 * S + 5, 2221 * S + 20), (0, S // 4, 0), (0, 0, 0), (K, 3, -K), 8, 5)
    ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, 0)
    ctx.tc_set_option(tc.TC_OPT_PRIORITY_BOOST, boost)
    got = {}
    for budget in (0, 60):
        ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, budget)
        print(budget, boost, flush=True)
        got[budget] = counted(ctx, F, Z, Z, [v], "budget %d" % budget)
    assert got[0] >= 200          # a cell at a time
    assert got[60] > got[0], got
