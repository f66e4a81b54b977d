"""Fewer loads than a plan holds: outer and inner iteration states of a mixed
solve lie at the plan's strides, not the call's.  Every load comes out as from
a plan of its own, bit for bit, whatever the plan solved before."""
import numpy as np
import pytest

from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import require_gpu

pytestmark = pytest.mark.gpu


# (96, 128, 96): large enough that two loads and more leave the queued phases
@pytest.mark.parametrize("shape,scheme", [((16, 24, 32), "cg"), ((6, 4, 12), "cg"), ((1, 32, 16), "cg"),
                                          ((96, 128, 96), "cg"), ((16, 24, 32), "basic"), ((6, 4, 12), "basic")])
def test_mixed_plan_solves_fewer_loads_than_it_holds(shape, scheme):
    require_gpu()
    print("case fewer loads", shape, scheme, flush=True)
    phase = M.random_phases(shape, 2, 3)
    lame = [[1.0, 0.7], [3.0, 5.0]]
    lam0, mu0 = M.midpoint_reference(lame)
    E = np.random.default_rng(8).uniform(-1, 1, (5, 6))
    if shape[0] == 1:
        E[:, [0, 4, 5]] = 0.0
    kw = dict(lame=lame, scheme=scheme, precision="mixed", tol=1e-9, max_iter=20000, autotune=False)
    ref = []
    for e in E:
        s = ffth.Solver(phase, lam0, mu0, nloads=1, **kw)
        eps, res = s.solve_order0(e[None])
        assert res[0]["status"] == 0 and res[0]["iters"] > 0
        ref.append((eps[0].cpu().numpy(), res[0]["iters"], res[0]["residual"]))
        s.close()
    s = ffth.Solver(phase, lam0, mu0, nloads=5, **kw)
    for loads in ([0, 1], [2], [0, 1, 2, 3, 4], [4, 3, 2], [1]):
        eps, res = s.solve_order0(E[loads])
        eps = eps.cpu().numpy()
        for i, l in enumerate(loads):
            assert res[i]["status"] == 0
            assert (res[i]["iters"], res[i]["residual"]) == ref[l][1:]
            assert np.array_equal(eps[i], ref[l][0])
    s.close()
