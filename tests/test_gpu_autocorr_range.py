"""Autocorrelation removal where taps and gains are of very different size but
their products, the weights, are ordinary."""
import dataclasses

import numpy as np
import pytest

import oracle
from coverage_layouts import box

pytestmark = pytest.mark.gpu

TOL = 1e-5   # the library's FP32 bar, on the full image


@pytest.fixture(scope="module")
def E():
    from paper_2301_09662_amd import epic
    return epic


@pytest.mark.parametrize("n_pol", [1, 2])
@pytest.mark.parametrize("size", [1e-25, 1e-20, 1e-3, 1.0, 3e7, 1e20, 1e25])
def test_gains_undo_the_taps(E, size, n_pol):
    import torch
    s = dataclasses.replace(box(32, 14, 12, P=n_pol, n_extra=9, seed=2), n_chan=2)
    rng = np.random.default_rng(5)
    x = rng.integers(0, 256, (6, 2, s.n_ant, n_pol), dtype=np.uint8)
    taps = (rng.standard_normal((2, s.n_ant, n_pol, 3, 3, 2)) * size).astype(np.float32)
    gains = (rng.standard_normal((2, s.n_ant, n_pol, 2)) / size).astype(np.float32)
    t = (taps[..., 0] + 1j * taps[..., 1].astype(np.float64)) * (
        gains[..., 0] + 1j * gains[..., 1].astype(np.float64))[..., None, None]
    w = np.stack([t.real, t.imag], axis=-1).astype(np.float32)
    out = torch.empty((2, 4 if n_pol == 2 else 1, 32, 32), device="cuda")
    plan = E.epic_plan([s], max_time=6, taps=[taps], flags=E.EPIC_F_REMOVE_AUTOCORR)
    try:
        E.epic_set_gains(plan, 0, gains)
        E.epic_grid_fft_accumulate(plan, [torch.from_numpy(x).cuda()], 6)
        E.epic_readout(plan, [out], 1)
        got = out.double().cpu().numpy()
    finally:
        E.epic_destroy(plan)
    full = oracle.image(s, x, taps=w)
    ref = full - oracle.autocorr(s, x, taps=w)
    assert np.isfinite(got).all()
    for c in range(2):
        assert np.abs(got[c] - ref[c]).max() <= TOL * np.abs(full[c]).max(), c
