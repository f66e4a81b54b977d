"""Which passes a plan runs for which tile variants: all 0, the passes it was
created with (grouped, or one spectral pass on a plane); others, the classical
passes with those tiles.  The y-pass launches of the kernel timing tell the
routes apart.  Writing back what was read changes nothing, bit for bit."""
import numpy as np
import pytest

from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import require_gpu, to_dev

pytestmark = pytest.mark.gpu


def _apply(torch, s, tau, precision):
    """Result and y-pass launches of one operator application."""
    ffth.ffth_profile_enable(s.plan, True)
    out = s.green_apply(tau, precision=precision).cpu().numpy()
    prof = ffth.ffth_profile_read(s.plan)
    ffth.ffth_profile_enable(s.plan, False)
    return out, prof["ypass_f64" if precision == "fp64" else "ypass_f32"][0]


@pytest.mark.parametrize("shape", [(16, 24, 32), (8, 96, 12), (1, 48, 16), (1, 512, 8)])
def test_variants_written_back_change_nothing(shape):
    torch = require_gpu()
    print("case variants written back", shape, flush=True)
    tau = to_dev(torch, np.random.default_rng(sum(shape)).standard_normal((6,) + shape))
    s = ffth.Solver(np.zeros(shape, np.uint16), 1.4, 0.9, lame=[[2.0, 1.0]], autotune=False)
    own = {}
    for precision in ("fp64", "fp32"):
        own[precision], y = _apply(torch, s, tau, precision)
        assert y == 0
    s.tile_variants = s.tile_variants
    for precision in ("fp64", "fp32"):
        got, y = _apply(torch, s, tau, precision)
        assert y == 0 and np.array_equal(got, own[precision])
    for pin, y64, y32 in (([4] * 8, 2, 2), ([0, 4] * 4, 2, 0 if shape[0] > 1 else 2)):
        s.tile_variants = pin
        assert _apply(torch, s, tau, "fp64")[1] == y64 and _apply(torch, s, tau, "fp32")[1] == y32
        s.tile_variants = [0] * 8
        for precision in ("fp64", "fp32"):
            got, y = _apply(torch, s, tau, precision)
            assert y == 0 and np.array_equal(got, own[precision])
    s.close()


def test_plane_keeps_its_single_pass_with_other_tiles():
    """The tuner's variants of a plane (no y shape) stand for its one-pass step."""
    torch = require_gpu()
    shape = (1, 64, 32)
    tau = to_dev(torch, np.random.default_rng(3).standard_normal((6,) + shape))
    s = ffth.Solver(np.zeros(shape, np.uint16), 1.4, 0.9, lame=[[2.0, 1.0]], autotune=False)
    ref, _ = _apply(torch, s, tau, "fp64")
    for v in range(1, ffth.TILE_VARIANTS):
        s.tile_variants = [v, v, 0, 0, v, v, v, v]
        got, y = _apply(torch, s, tau, "fp64")
        assert y == 0
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max(), v   # rounding only
    s.close()
