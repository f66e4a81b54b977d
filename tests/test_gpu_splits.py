"""Iteration kernels of every split of axis 1 (n1 = R1 R2) that a grid can
take, in each precision and material kind, against the classical passes (a
plan with tile variants other than 0 runs those): solves to residual 1e-10
agree to 2e-8, as each is within 1e-10 of the solution in residual, times at
most the stiffness contrast (about 10) in the field."""
import numpy as np
import pytest

from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import rel_l2, require_gpu

pytestmark = pytest.mark.gpu

# (R1, R2) in FP32; in FP64
SHAPES = [(8, 8, 8),        # 2, 4;  2, 4
          (8, 12, 16),      # 2, 6;  3, 4
          (24, 16, 8),      # 2, 8;  4, 4
          (8, 24, 8),       # 4, 6;  6, 4
          (8, 32, 8),       # 4, 8;  8, 4
          (16, 48, 16),     # 8, 6; 12, 4
          (8, 64, 8),       # 8, 8;  8, 8
          (8, 96, 12),      # 16, 6; 12, 8
          (12, 128, 16),    # 16, 8; 16, 8
          (8, 256, 8),      # 16, 16; 16, 16
          # second choices: the preferred R2's tile does not fit a long axis 0
          (256, 8, 8),      # 2, 4;  4, 2
          (256, 12, 8),     # -;     6, 2
          (256, 16, 8),     # 4, 4;  8, 2
          (256, 24, 8),     # -;    12, 2
          (256, 32, 8),     # 8, 4; 16, 2
          (128, 64, 8),     # 8, 8; 16, 4
          (256, 64, 8)]     # 16, 4; -
WIDE = [(256, 128, 64),     # 32, 4; -
        (96, 256, 64)]      # 32, 8; -

LAME = [[1.0, 0.7], [4.0, 2.0], [0.8, 6.0]]


def _triclinic(seed):
    """Three positive definite stiffness matrices with 21 independent entries,
    eigenvalues in [2, 8] before the shear rows' scale."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(3):
        q, _ = np.linalg.qr(rng.standard_normal((6, 6)))
        c = q @ np.diag(rng.uniform(2.0, 8.0, 6)) @ q.T
        out.append(c[np.triu_indices(6)])
    return np.array(out)


def _both_routes(shape, general, **opts):
    phase = M.random_phases(shape, 3, sum(shape))
    mat = dict(voigt21=_triclinic(7)) if general else dict(lame=LAME)
    lam0, mu0 = (2.0, 2.5) if general else M.midpoint_reference(LAME)
    E = np.random.default_rng(1).uniform(-1, 1, (2, 6))
    out = []
    for pinned in (False, True):
        s = ffth.Solver(phase, lam0, mu0, nloads=2, tol=1e-10, autotune=False, **mat, **opts)
        if pinned:
            s.tile_variants = [4] * 8
        ffth.ffth_profile_enable(s.plan, True)
        eps, res = s.solve_order0(E)
        prof = ffth.ffth_profile_read(s.plan)
        assert all(r["status"] == 0 for r in res)
        out.append((eps.cpu().numpy(), np.array([r["mean_stress"] for r in res]),
                    prof["ypass_f32"][0], prof["ypass_f64"][0]))
        s.close()
    for i in range(2):
        assert rel_l2(out[0][0][i], out[1][0][i]) < 2e-8
    assert np.abs(out[0][1] - out[1][1]).max() < 2e-8 * np.abs(out[1][1]).max()
    return out[0][2:], out[1][2:]


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("scheme,precision,h16", [("cg", "mixed", False), ("cg", "mixed", "force"),
                                                  ("cg", "fp64", False), ("cg3", "fp64", False),
                                                  ("bicgstab", "fp64", False)])
@pytest.mark.parametrize("shape", SHAPES)
def test_iteration_kernels_of_every_split(shape, scheme, precision, h16, general):
    require_gpu()
    print("case split", shape, scheme, precision, h16, general, flush=True)
    own, pinned = _both_routes(shape, general, scheme=scheme, precision=precision, spectrum16=h16)
    assert pinned[1] > 0 and (precision == "fp64" or pinned[0] > 0)
    if shape not in ((256, 12, 8), (256, 24, 8)):      # FP32 has no split that fits these
        assert own[0] == 0
    if shape != (256, 64, 8):                          # nor FP64 this one
        assert own[1] == 0


@pytest.mark.parametrize("h16,general", [(False, False), ("force", False), ("force", True)])
@pytest.mark.parametrize("shape", WIDE)
def test_iteration_kernels_of_wide_groups(shape, h16, general):
    require_gpu()
    print("case split", shape, h16, general, flush=True)
    own, pinned = _both_routes(shape, general, scheme="cg", precision="mixed", spectrum16=h16)
    assert own[0] == 0 and pinned[0] > 0
