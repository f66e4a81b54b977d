"""Every z-tile variant on axes of 512 and 1024 points, where the FP64 shapes
differ in columns and threads, against the FP64 oracle (rounding only: 1e-12 in
FP64, 5e-6 in FP32, as for the shorter axes)."""
import numpy as np
import pytest

from oracle import spectral
from paper_1712_05145_amd import ffth
from tests._gpu import full, rel_l2, require_gpu, to_dev, voigt6

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", range(6))
@pytest.mark.parametrize("shape", [(512, 6, 4), (1024, 4, 6), (1, 512, 8), (1, 1024, 4)])
def test_z_tiles_of_long_axes(variant, shape):
    torch = require_gpu()
    print("case long axis tile", variant, shape, flush=True)
    tau = np.random.default_rng(7 + sum(shape)).standard_normal((6,) + shape)
    ref = voigt6(spectral.green_apply(full(tau), 1.7, 0.9))
    s = ffth.Solver(np.zeros(shape, np.uint16), 1.7, 0.9, lame=[[2.0, 1.0]], autotune=False)
    s.tile_variants = [0, 0, 0, 0, variant, variant, 0, 0]
    for precision, tol in (("fp64", 1e-12), ("fp32", 5e-6)):
        got = s.green_apply(to_dev(torch, tau), precision=precision).cpu().numpy()
        assert rel_l2(got, ref) < tol, (precision, rel_l2(got, ref))
    s.close()
