"""Autocorrelation removal when the caller captures calls without running them:
a gain change folds the zero-lag sums gathered before it under the gains that
they were gathered with, whatever the host had counted by then."""
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


@pytest.mark.parametrize("captured", ["gains", "readout"])
def test_gain_change_folds_what_is_pending(E, captured):
    """Five spectra under gains g, five under unit gains.  The change is either
    replayed from a graph captured when nothing was pending, or made eagerly
    after a read-out that was captured and not run."""
    import torch
    s = dataclasses.replace(box(32, 14, 12, n_extra=9, seed=2), n_chan=3)
    rng = np.random.default_rng(1)
    x = rng.integers(0, 256, (2, 5, 3, s.n_ant, 2), dtype=np.uint8)
    d = [torch.from_numpy(v).cuda() for v in x]
    g = np.zeros((3, s.n_ant, 2, 2), np.float32)
    g[..., 0] = rng.uniform(0.5, 2.0, (3, s.n_ant, 1))
    out, unused = (torch.empty((3, 4, 32, 32), device="cuda") for _ in range(2))
    plan = E.epic_plan([s], max_time=5, flags=E.EPIC_F_REMOVE_AUTOCORR)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    try:
        E.epic_set_gains(plan, 0, g)
        if captured == "readout":
            E.epic_grid_fft_accumulate(plan, [d[0]], 5)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            if captured == "gains":
                E.epic_set_gains(plan, 0, None, side)
            else:
                E.epic_readout(plan, [unused], 0, side)
        if captured == "gains":
            E.epic_grid_fft_accumulate(plan, [d[0]], 5)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
        else:
            E.epic_set_gains(plan, 0, None)
        E.epic_grid_fft_accumulate(plan, [d[1]], 5)
        E.epic_readout(plan, [out], 1)
        got = out.double().cpu().numpy()
    finally:
        E.epic_destroy(plan)
    t = oracle.taps(s) * g[..., 0][..., None, None]
    taps = np.stack([t.real, t.imag], axis=-1).astype(np.float32)
    full = oracle.image(s, x[0], taps=taps) + oracle.image(s, x[1])
    ref = full - oracle.autocorr(s, x[0], taps=taps) - oracle.autocorr(s, x[1])
    for c in range(3):
        assert np.abs(got[c] - ref[c]).max() <= TOL * np.abs(full[c]).max(), c
