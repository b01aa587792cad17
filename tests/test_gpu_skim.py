"""The single-precision walk against the oracle where its rounded values
cannot decide: rays through lattice corners and along cell lines, heights on
and one unit beside a column's own height, and origins as far from the map
as the boundary accepts.  Hit words are whole numbers and must be equal;
depths are the oracle's, rounded once (1e-6 relative)."""
import numpy as np
import pytest

import oracle
from synth.views import VIEW_DTYPE

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_parity import load  # noqa: E402

S = 65536
W, H = 93, 61


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    c = tc.Context(0)
    yield c
    c.close()


def terrain():
    """Plateaus at a few heights (so that rays meet tops at their own height)
    under slabs, and one wall on every side of the middle."""
    rng = np.random.default_rng(5)
    F = np.kron(rng.choice([0, 7, 8, 20, 60], (H // 8 + 1, W // 8 + 1)), np.ones((8, 8)))
    F = F[:H, :W].astype(np.uint8)
    two = np.kron(rng.random((H // 4 + 1, W // 4 + 1)) < 0.3, np.ones((4, 4)))[:H, :W] > 0
    B = np.where(two, F.astype(int) + rng.choice([1, 5, 40], (H, W)), 0)
    T = np.where(two, np.minimum(B + rng.choice([0, 3], (H, W)), 255), 0)
    return F, B.astype(np.uint8), T.astype(np.uint8)


def ortho(o0, o_px, o_py, d, w, h):
    v = np.zeros((), VIEW_DTYPE)
    v["width"], v["height"] = w, h
    v["o0"], v["o_px"], v["o_py"], v["d0"] = o0, o_px, o_py, d
    return v


def views(kind):
    out = []
    if kind == "corners":          # every crossing a corner or a near miss of one
        for a, b in ((1, 1), (1, -1), (2, 1), (-1, 3), (-3, -2), (1, 0), (0, -1)):
            for off in (0, 1, -1):
                k = (1 << 22) // 6
                o = (off, 0, 30 * S) if a >= 0 else (W * S + off, 0, 30 * S)
                if b < 0:
                    o = (o[0], H * S, o[2])
                out.append(ortho(o, (S // 2, 0, 0), (0, S // 2, 0), (a * k, b * k, -k // 40), 40, 24))
    elif kind == "levels":         # level rays on and beside whole heights
        for a, b in ((5, 1), (-2, 7), (1, 0), (0, 1)):
            for z in (7 * S, 7 * S + 1, 8 * S - 1, 8 * S, 8 * S + 3, 60 * S):
                k = (1 << 22) // 7
                out.append(ortho((40 * S + 9, 30 * S + 5, z), (S // 2 + 3, 0, 0), (0, S // 2 + 1, 0),
                                 (a * k, b * k, 0), 17, 9))
    elif kind == "shallow":        # a fall of one unit over many cells
        for dz in (-1, 1, -2):
            for z in (8 * S + 1, 20 * S, 20 * S + 1):
                out.append(ortho((0, 3, z), (0, 0, 0), (0, S // 2, 0), (1 << 22, 77, dz * 70), 3, 60))
                out.append(ortho((W * S - 1, 3, z), (0, 0, 0), (0, S // 2, 0), (-(1 << 22), 1, dz), 3, 60))
    else:                          # far: origins near the ends of their range
        for sx in (-1, 1):
            for sz in (-1, 1):
                far = 32000
                x, z = sx * far, (far if sz > 0 else -200)
                k = 1 << 22
                d = (-sx * k, 0, -int(k * (z - 20) / (far - (W if sx > 0 else 0))))
                out.append(ortho((x * S, 7, z * S), (0, 0, 64), (0, S // 2, 0), d, 20, 58))
                out.append(ortho((x * S, 7 - 16000 * S, z * S), (0, 0, 64), (0, S // 2, 0),
                                 (d[0], k // 2, d[2]), 20, 58))
    return out


@pytest.mark.parametrize("kind", ["corners", "levels", "shallow", "far"])
@pytest.mark.parametrize("beam,split,boost", [(0, 0, 0), (6, 120, 0), (6, 3, 0), (6, 40, 5)])
def test_skim(ctx, kind, beam, split, boost):
    F, B, T = terrain()
    load(ctx, F, B, T)
    vs = views(kind)
    ctx.tc_set_option(tc.TC_OPT_BEAM_PASSES, beam)
    ctx.tc_set_option(tc.TC_OPT_SPLIT_BUDGET, split)
    ctx.tc_set_option(tc.TC_OPT_PRIORITY_BOOST, boost)
    print(kind, beam, split, len(vs), flush=True)
    wo, do = oracle.render(F, B, T, vs)
    out = tc.render(ctx, vs)
    torch.cuda.synchronize()
    wg, dg = tc.split_hits(out)
    assert np.array_equal(wg, wo), np.count_nonzero(wg != wo)
    hit = wo != oracle.MISS
    assert hit.any()
    np.testing.assert_allclose(dg[hit], do[hit], rtol=1e-6)
    assert np.isinf(dg[~hit]).all()
