"""bench.py's byte models against the streams of the passes that run: grouped
grids have no y-passes, a solve's first passes read no iterate, field passes
read no phase ids.  CPU only."""
import bench

F32, F64, H16, IDS = 24.0, 48.0, 12.0, 2.0


def test_grouped_inner_iteration_has_no_y_passes():
    m16, m32 = bench.alg_bytes_per_voxel(True, grouped=True), bench.alg_bytes_per_voxel(False, grouped=True)
    assert m16["xcg3"] + m16["yf"] + m16["z"] + m16["yi"] == 158.0 + H16 + F32      # 194, classical 266
    assert m32["xcg3"] + m32["yf"] + m32["z"] + m32["yi"] == 170.0 + F32 + F32      # 218, classical 314
    m = bench.inner_models(m16, 1000, 50, 3, 7)
    assert m["ypass_f32"] == 0.0
    assert m["zpass_f32"] == 1000 * (50 * (H16 + F32) + 3 * (F32 + F32))
    m = bench.inner_models(bench.alg_bytes_per_voxel(True), 1000, 50, 3, 7)
    assert m["ypass_f32"] == 1000 * (50 * (H16 + H16 + F32 + F32) + 3 * 2 * (F32 + F32))
    assert m["xcg3_f32"] == 1000 * (50 * 158.0 - 7 * bench.XCG3_START_SAVING)


def test_mixed_sweeps_read_the_iterate_from_the_third_on():
    def xf(sweeps):
        rec = {"iters": 0, "fp64_applications": sweeps, "projections": 0}
        return bench.mixed_fp64_models([[rec]], 1, order1_index=-1)["xfwd_f64"]
    # sweep 1: ids, spectrum out; 2: ids, correction, iterate and spectrum out; 3: the iterate read as well
    assert xf(2) - xf(1) == IDS + F32 + F64 + F64
    assert xf(3) - xf(2) == IDS + F32 + F64 + F64 + F64
    # right-hand side of order 1: six fields (6 components in) and one of 3, spectra out; no ids
    assert xf(1) == IDS + F64 + 6 * (F64 + F64) + (24.0 + F64)


def test_first_application_reads_no_iterate():
    rec = {"iters": 0, "fp64_applications": 2, "projections": 0}
    rhs_xf, rhs_xi = 6 * (F64 + F64) + 24.0 + F64, 6 * (F64 + 24.0) + 3 * F64
    m = bench.fp64_models([[rec]], 1, "cg", order1_index=-1)
    assert m["xfwd_f64"] == rhs_xf + (IDS + F64) + (IDS + F64 + F64)
    assert m["xinv_f64"] == rhs_xi + (F64 + F64) + (F64 + F64 + F64)
    m = bench.fp64_models([[rec]], 1, "cg3", order1_index=-1)
    assert m["xfwd_f64"] == rhs_xf + IDS + F64
    assert m["xinv_f64"] == rhs_xi + F64 + F64
