"""Shadow rays in the cell they start in: one unit off tops, undersides and
walls, under thin and zero-thickness slabs, along cell lines and through
corners, level, steep and from below.  RGBA bit for bit the oracle's."""
import pytest

import oracle
import synth

tc = pytest.importorskip("paper_2608_17390_amd")
torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_shade import assert_same, gpu_shade, load  # noqa: E402
from test_gpu_skim import H, W, S, ortho, terrain  # noqa: E402

K = 1 << 20
LIGHTS = [(K, 0, 0), (0, -K, 1), (K, K, K), (-K, 2 * K, 3), (3, -1, K), (K, K // 3, -K // 5),
          (-1, 0, -K), (0, 0, K), (5, 0, -3)]


@pytest.mark.parametrize("light", LIGHTS)
def test_shadow(light):
    F, B, T = terrain()
    d = 1 << 21
    vs = [ortho((0, 0, 270 * S), (S // 2, 0, 0), (0, S // 2, 0), (0, 0, -d), W, H),
          ortho((0, 0, 270 * S), (S // 2, 0, 0), (0, S // 2, 0), (d // 7, -d // 3, -d), W, H),
          # along the ground from each side, and up against the undersides
          ortho((0, 0, 9 * S), (0, S // 2, 0), (0, 0, S // 3), (d, 3, 0), H, 40),
          ortho((W * S - 1, 0, S), (0, S // 2, 0), (0, 0, S // 3), (-d, d // 50, d // 400), H, 60),
          synth.perspective_view((W / 2 + 0.5, -20.0, 30.0), 0, -8, 61, 33)]
    with tc.Context(0) as ctx:
        load(ctx, F, B, T)
        pal = synth.default_palette()
        print(light, flush=True)
        assert_same(gpu_shade(ctx, vs, light, pal), oracle.shade(F, B, T, vs, light, pal), str(light))
