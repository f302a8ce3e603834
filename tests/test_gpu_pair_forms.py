"""Every compiled window size of the paired-transform kernel with either number
of pols, and which plans run that kernel."""
import dataclasses

import numpy as np
import pytest

import oracle
from coverage_layouts import box
from gpu_util import assert_parity, run_library

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp16": 1e-3}   # the library's bars per image
GRIDS = (32, 48, 64, 96, 128, 192, 256)
# (W, R): each compiled size 8, 16, 20, 24, 32, 40, 48, 52, 64 as its smallest and largest window
WINDOWS = [(4, 8), (8, 7), (9, 16), (20, 17), (21, 24), (24, 25), (32, 29), (33, 32), (40, 36), (41, 33), (48, 45), (49, 52),
           (53, 49), (57, 64), (64, 5)]


@pytest.fixture(scope="module")
def E():
    from paper_2301_09662_amd import epic
    return epic


@pytest.mark.parametrize("precision", ["fp32", "fp16"])
@pytest.mark.parametrize("n_pol", [1, 2])
@pytest.mark.parametrize("N", GRIDS)
def test_every_window_and_pol_count(E, N, n_pol, precision):
    subs = [box(N, W, R, P=n_pol, n_extra=7, seed=3 * N + k) for k, (W, R) in enumerate(WINDOWS) if max(W, R) <= N]
    rng = np.random.default_rng(N)
    xs = [rng.integers(0, 256, (3, 1, s.n_ant, n_pol), dtype=np.uint8) for s in subs]
    gpus, info = run_library(E, subs, xs, precision=precision)
    for s, x, g in zip(subs, xs, gpus):
        assert_parity(g, oracle.image(s, x), TOL[precision], f"{precision} N={N} P={n_pol} window {s.W}x{s.R}")
