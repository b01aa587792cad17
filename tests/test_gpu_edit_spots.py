"""Many edits of one place: craters of every size and depth over patches and
under them, rectangles as large and as far as they may be, up to the longest
list that goes block by block; against a fresh load of the oracle's map.  And
such a list against the next longer one, whose cells are updated in a launch
of their own: going through a block's edits must not take several times as
long."""
import numpy as np
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_edit_tiles import crater, levels  # noqa: E402


def patch(rng, x, y, w, h):
    F = rng.integers(0, 200, (h, w)).astype(np.uint8)
    B = np.where(rng.random((h, w)) < 0.4, F + rng.integers(1, 40, (h, w)), 0).astype(np.uint8)
    T = np.where(B > 0, B + rng.integers(0, 10, (h, w)), 0).astype(np.uint8)
    return dict(kind=1, x0=x, y0=y, w=w, h=h, F=F, B=B, T=T)


def lists(W, H):
    rng = np.random.default_rng(W + 7 * H)
    yield "sizes", [crater(int(rng.integers(-s, W)), int(rng.integers(-s, H)), s, int(d))
                    for s in (1, 2, 3, 16, 63, 64, 65, 255, 256, 1000, 2047, 2048, 4095, 4096)
                    for d in (0, 1, 2, 128, 255)]
    yield "layers", [patch(rng, int(rng.integers(-9, W)), int(rng.integers(-9, H)), int(rng.integers(1, 40)),
                           int(rng.integers(1, 40))) if k % 3 else
                     crater(int(rng.integers(-9, W)), int(rng.integers(-9, H)), int(rng.integers(1, 50)),
                            int(rng.integers(0, 40))) for k in range(300)]
    far = (1 << 31) - 1
    yield "far", [crater(far - 4096, far - 4096, 4096, 255), crater(-(1 << 28), -(1 << 28), 4096, 255),
                  crater(far - 3, 0, 3, 9), patch(rng, -(1 << 28), 0, 5, 5), crater(W - 1, H - 1, 4096, 3),
                  crater(-4095, -4095, 4096, 200), patch(rng, W - 2, -3, 7, 9)]
    yield "one spot", [crater(W // 3 + k % 9, H // 3 + k % 7, 8 + k % 90, 1 + k % 3) for k in range(512)]
    yield "saturated", [crater(W // 3 - 20, H // 3 - 20, 60, 255) for _ in range(512)]


@pytest.mark.parametrize("W,H", [(50, 40), (130, 67), (700, 333)])
def test_edit_spots(W, H):
    F, B, T = synth.make_map(W, H, 70 + W, dual=0.3, period=8)
    with tc.Context(0) as ctx, tc.Context(0) as fresh:
        for name, edits in lists(W, H):
            print(W, H, name, flush=True)
            ctx.tc_load_columns(F, B, T)
            ctx.tc_apply_edit(edits)
            fresh.tc_load_columns(*oracle.apply_edits(F, B, T, edits))
            for (what, got), (_, want) in zip(levels(ctx), levels(fresh)):
                assert np.array_equal(got, want), (name, what)


@pytest.mark.parametrize("size,area", [(16, 24), (32, 100)])
def test_edit_spot_time(size, area):
    F = np.full((1024, 1024), 200, np.uint8)
    Z = np.zeros_like(F)
    rng = np.random.default_rng(3)
    edits = [crater(500 + int(rng.integers(0, area)), 500 + int(rng.integers(0, area)), size, 1)
             for _ in range(513)]
    v = [synth.perspective_view((100.5, 100.5, 260.0), 0, -60, 8, 8)]
    out = torch.empty((64, 2), dtype=torch.int32, device="cuda")
    ms = {512: [], 513: []}
    with tc.Context(0) as ctx:
        ctx.tc_load_columns(F, Z, Z)
        frames = {n: ctx.tc_frame_create(v, edits[:n], out.data_ptr()) for n in ms}
        for _ in range(15):
            for n, f in frames.items():
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                f.launch()
                b.record()
                b.synchronize()
                ms[n].append(a.elapsed_time(b))
        for f in frames.values():   # (before the context)
            f.close()
    short, longer = (np.median(ms[n][3:]) for n in (512, 513))
    print(size, area, short, longer, flush=True)
    assert short <= 1.5 * longer, (short, longer)
