"""GPU parity of the grouped passes (axis 1 split between the x-passes and the
z-pass) and of the one-pass spectral step of 2-D grids against the FP64
oracle, over the axis lengths whose splits differ and the edges of their
tiles, and against the classical five passes, which a plan with pinned tile
shapes runs.

Tolerances: FP64 operator applications 1e-12 relative L2 and FP32 ones 5e-6,
as for the classical passes (rounding only).  Solves to residual 1e-10 agree
to 2e-8 between the routes: each is within 1e-10 of the solution in residual,
times at most the stiffness contrast in the field.  Finalizes carried by a
pass do the sums of a separate launch in the same order, so iterates do not
depend, bit for bit, on how often the host reads the states."""
import ctypes

import numpy as np
import pytest

from oracle import spectral
from paper_1712_05145_amd import ffth
from paper_1712_05145_amd import microstructure as M
from tests._gpu import full, rel_l2, require_gpu, to_dev, voigt6

pytestmark = pytest.mark.gpu

# every split of axis 1, the smallest and largest lengths of the other axes,
# blocks with a ragged last group, and lengths just outside the rule
SHAPES = [(8, 8, 8), (12, 12, 24), (8, 16, 12), (24, 24, 8), (8, 32, 16), (12, 48, 8), (16, 64, 8), (8, 96, 12),
          (8, 128, 8), (128, 8, 8), (96, 12, 16), (128, 24, 12), (8, 16, 256), (8, 64, 256), (12, 12, 128),
          (64, 32, 96), (1, 12, 16), (1, 48, 96), (1, 256, 8),
          # axes of 256, both choices of the split, and lengths the rule leaves out
          (8, 256, 8), (64, 256, 32), (96, 256, 64), (64, 256, 16), (256, 8, 12), (256, 32, 8), (256, 64, 32),
          (256, 128, 64), (256, 24, 16), (48, 256, 96), (128, 64, 96), (64, 128, 64)]


@pytest.mark.parametrize("shape", SHAPES)
def test_green_operator_every_split(shape):
    torch = require_gpu()
    print("case grouped green", shape, flush=True)
    tau = np.random.default_rng(sum(shape)).standard_normal((6,) + shape)
    ref = voigt6(spectral.green_apply(full(tau), 1.4, 0.9))
    s = ffth.Solver(np.zeros(shape, np.uint16), 1.4, 0.9, lame=[[2.0, 1.0]], autotune=False)
    for precision, tol in (("fp64", 1e-12), ("fp32", 5e-6)):
        got = s.green_apply(to_dev(torch, tau), precision=precision).cpu().numpy()
        assert rel_l2(got, ref) < tol, (precision, rel_l2(got, ref))
    s.tile_variants = [0] * 8     # the classical passes
    for precision, tol in (("fp64", 1e-12), ("fp32", 5e-6)):
        got = s.green_apply(to_dev(torch, tau), precision=precision).cpu().numpy()
        assert rel_l2(got, ref) < tol, (precision, rel_l2(got, ref))


@pytest.mark.parametrize("shape", [(8, 12, 16), (24, 16, 8), (16, 48, 32), (12, 128, 16), (1, 24, 32), (8, 256, 16),
                                   (256, 16, 8)])
@pytest.mark.parametrize("scheme,precision,h16", [("cg", "mixed", False), ("cg", "mixed", "force"),
                                                  ("basic", "mixed", False), ("cg", "fp64", False),
                                                  ("cg3", "fp64", False), ("bicgstab", "fp64", False)])
def test_solves_agree_with_classical_passes(shape, scheme, precision, h16):
    torch = require_gpu()
    print("case grouped solve", shape, scheme, precision, h16, flush=True)
    phase = M.random_phases(shape, 3, 5)
    lame = [[1.0, 0.7], [4.0, 2.0], [0.8, 6.0]]
    lam0, mu0 = M.midpoint_reference(lame)
    E = np.random.default_rng(1).uniform(-1, 1, (2, 6))
    if shape[0] == 1:
        E[:, [0, 4, 5]] = 0.0
    out = []
    for pinned in (False, True):
        s = ffth.Solver(phase, lam0, mu0, lame=lame, nloads=2, scheme=scheme, precision=precision, tol=1e-10,
                        autotune=False, spectrum16=h16)
        if pinned:
            s.tile_variants = [0] * 8
        eps, res = s.solve_order0(E)
        assert all(r["status"] == 0 for r in res)
        out.append((eps.cpu().numpy(), np.array([r["mean_stress"] for r in res])))
        s.close()
    for i in range(2):
        assert rel_l2(out[0][0][i], out[1][0][i]) < 2e-8
    assert np.abs(out[0][1] - out[1][1]).max() < 2e-8 * np.abs(out[1][1]).max()


@pytest.mark.parametrize("shape", [(8, 12, 24), (24, 48, 8), (8, 96, 12), (6, 4, 12), (4, 6, 1024), (1, 16, 48),
                                   (1, 6, 4)])
def test_field_passes(shape):
    """Field in, field out without a solve: six components out of three values
    per pass (displacement) and the allocation-free operator, over grouped and
    classical plans with ragged last blocks; input and output may be one array."""
    torch = require_gpu()
    print("case field passes", shape, flush=True)
    rng = np.random.default_rng(sum(shape))
    tau = rng.standard_normal((6,) + shape)
    s = ffth.Solver(np.zeros(shape, np.uint16), 1.1, 0.6, lame=[[2.0, 1.0]], autotune=False)
    ref = spectral.displacement_from_strain(full(tau))
    assert rel_l2(s.displacement(to_dev(torch, tau)).cpu().numpy(), ref) < 1e-12
    ref = voigt6(spectral.green_apply(full(tau), 1.1, 0.6))
    for precision, tol in (("fp64", 1e-12), ("fp32", 5e-6)):
        a = to_dev(torch, tau)
        ffth.ffth_green_apply_noalloc(shape, 1.1, 0.6, ffth._dptr(a), ffth._dptr(a), ffth.PRECISIONS[precision],
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rel_l2(a.cpu().numpy(), ref) < tol


@pytest.mark.parametrize("shape", [(16, 24, 32), (1, 32, 16)])
@pytest.mark.parametrize("scheme,precision", [("cg", "mixed"), ("cg3", "fp64"), ("cg", "fp32")])
def test_carried_finalize_bit_identical(shape, scheme, precision):
    """check_every = 1 gives every finalize a launch of its own; 7 lets six of
    seven ride in the next spectral step."""
    torch = require_gpu()
    print("case carried finalize", shape, scheme, precision, flush=True)
    phase = M.random_phases(shape, 2, 3)
    lame = [[1.0, 0.7], [3.0, 5.0]]
    lam0, mu0 = M.midpoint_reference(lame)
    E = np.array([[0.0, 1.0, -0.5, 0.3, 0.0, 0.0]])
    got = []
    for check in (1, 7):
        s = ffth.Solver(phase, lam0, mu0, lame=lame, scheme=scheme, precision=precision,
                        tol=1e-5 if precision == "fp32" else 1e-10, check_every=check, autotune=False)
        eps, res = s.solve_order0(E)
        assert res[0]["status"] == 0
        got.append((eps.cpu().numpy(), res[0]["iters"]))
        s.close()
    assert got[0][1] == got[1][1]
    assert np.array_equal(got[0][0], got[1][0])
