"""The benchmark's count of executed matrix products knows which FP32 plans run
the paired-transform kernel: at N = 128 and 192 its workgroups differ in size from
those of the vector kernel."""
import pytest

import bench
from coverage_layouts import box

THREADS = {128: 512, 192: 768}   # of the paired-transform kernel


@pytest.mark.parametrize("N,W,R,n_pol,n_ant", [
    (128, 20, 18, 2, 30), (128, 64, 64, 1, 30), (128, 64, 64, 2, 30), (128, 53, 53, 2, 900), (128, 60, 60, 2, 900),
    (128, 57, 57, 2, 2500), (128, 40, 40, 2, 2500), (192, 52, 50, 2, 30), (192, 53, 20, 2, 30), (192, 64, 60, 1, 30)])
def test_paired_or_vector(N, W, R, n_pol, n_ant):
    from paper_2301_09662_amd import epic as E
    s = box(N, W, R, P=n_pol, n_extra=n_ant - 2, seed=W + n_ant)
    plan = E.epic_plan([s], max_time=4, flags=E.EPIC_F_DRY_RUN)
    try:
        info, g = E.epic_plan_query(plan), E.epic_debug_geometry(plan, 0)
        ext = -(-max(W, R) // 4) * 4
        wd = next(w for w in (8, 20, 32, 40, 52, 64) if w >= ext)
        paired = info["threads"][0] == THREADS[N]
        assert bench.paired_fp32(s, g, wd) == paired
        assert (bench.mfma_ops_per_spectrum(plan, [s]) > 0) == paired
    finally:
        E.epic_destroy(plan)
