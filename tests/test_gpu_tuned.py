"""Tuned tile shapes on grids whose passes have some to choose from: classical
in both precisions (axis 0 of length 6 has no grouped passes) and planes, whose
one spectral pass has shapes of its own.  The tuned solve agrees with the
default tiles (same operator, reductions in another order), and another plan
given the tuned variants does the same, bit for bit."""
import numpy as np
import pytest

from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(6, 256, 256), (6, 512, 96), (1, 512, 512), (1, 1024, 256)])
@pytest.mark.parametrize("precision,scheme", [("mixed", "cg"), ("fp64", "cg")])
def test_tuned_plan_matches_default_tiles(shape, precision, scheme):
    require_gpu()
    print("case tuned", shape, precision, flush=True)
    phase = M.random_phases(shape, 3, 2)
    lame = [[1.0, 0.7], [4.0, 2.0], [0.8, 6.0]]
    lam0, mu0 = M.midpoint_reference(lame)
    E = np.random.default_rng(5).uniform(-1, 1, (2, 6))
    if shape[0] == 1:
        E[:, [0, 4, 5]] = 0.0
    assert phase.size >= 64 ** 3
    out, tuned = {}, None
    for kind in ("tuned", "copied", "default"):
        s = ffth.Solver(phase, lam0, mu0, lame=lame, nloads=2, precision=precision, scheme=scheme, tol=1e-10,
                        autotune=kind == "tuned")
        if kind == "tuned":
            tuned = s.tile_variants, s.launch_loads
            print("variants", *tuned, flush=True)
            assert len(tuned[0]) == 8 and all(0 <= v < ffth.TILE_VARIANTS for v in tuned[0])
            if shape[0] == 1:
                assert tuned[0][2] == tuned[0][3] == 0
        elif kind == "copied":
            s.tile_variants, s.launch_loads = tuned
        else:
            assert s.tile_variants == [0] * 8
        ffth.ffth_profile_enable(s.plan, True)
        eps, res = s.solve_order0(E)
        prof = ffth.ffth_profile_read(s.plan)
        assert (prof["ypass_f64"][0] > 0) == (shape[0] > 1)      # classical, or the plane's single pass
        assert all(r["status"] == 0 for r in res)
        out[kind] = eps.cpu().numpy(), np.array([r["mean_stress"] for r in res])
        s.close()
    assert np.array_equal(out["copied"][0], out["tuned"][0])
    assert np.abs(out["tuned"][1] - out["default"][1]).max() < 2e-8 * np.abs(out["default"][1]).max()
    scale = np.abs(out["default"][0]).max()
    assert np.sqrt(np.mean((out["tuned"][0] - out["default"][0]) ** 2)) < 2e-8 * scale
