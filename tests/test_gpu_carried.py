"""Finalizes carried by a spectral pass while loads of the same launch stop:
the block that finalizes a load clears its gating flag while that load's tile
blocks start.  With check_every = 1 every finalize is a launch of its own and
no flag changes under a pass; the iterates, iteration counts and residuals of
the other windows are the same bit for bit (the sums are taken in the same
order, so nothing may differ).  Planes of 512 and 1024 run FP64 spectral
passes of 512 threads, of which 256 sum."""
import numpy as np
import pytest

from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 512, 8), (1, 1024, 6), (1, 64, 16), (8, 16, 12), (24, 8, 32)])
@pytest.mark.parametrize("scheme,precision", [("cg3", "fp64"), ("cg", "fp64"), ("cg", "mixed")])
def test_loads_that_stop_inside_a_window(shape, scheme, precision):
    torch = require_gpu()
    print("case carried finalize, stopping loads", shape, scheme, precision, flush=True)
    phase = M.random_phases(shape, 3, 11)
    lame = [[1.0, 0.7], [3.0, 5.0], [0.5, 1.5]]
    lam0, mu0 = M.midpoint_reference(lame)
    E = np.random.default_rng(2).uniform(-1, 1, (4, 6))
    E[1] = 0.0                      # stops with its first pass
    E[2] = [1.0, 1.0, 1.0, 0, 0, 0]
    E[3] = [0, 0, 0, 1.0, 0, 0]
    if shape[0] == 1:
        E[:, [0, 4, 5]] = 0.0
    got = []
    for check in (1, 5, 64):
        s = ffth.Solver(phase, lam0, mu0, lame=lame, nloads=4, scheme=scheme, precision=precision, tol=1e-10,
                        check_every=check, autotune=False)
        eps, res = s.solve_order0(E)
        assert all(r["status"] == 0 for r in res)
        got.append((eps.cpu().numpy(), [(r["iters"], r["residual"], tuple(r["mean_stress"])) for r in res]))
        s.close()
    assert len({r[0] for r in got[0][1]}) > 1      # the loads do stop at different iterations
    for g in got[1:]:
        assert np.array_equal(g[0], got[0][0])
        if precision != "mixed":
            assert g[1] == got[0][1]
        else:                                      # iterations past a stop are not counted either
            assert [r[0] for r in g[1]] == [r[0] for r in got[0][1]]
