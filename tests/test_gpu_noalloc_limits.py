"""epic_image_noalloc near its buffer's limit: whatever number of workgroups a
full launch has, a call whose images fit with two slots per channel runs."""
import dataclasses

import numpy as np
import pytest

from coverage_layouts import box
from gpu_util import assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_2301_09662_amd import epic
    return epic


# (precision, gridder, N, P, antennas, channels, spectra)
CASES = [("fp16", "auto", 64, 2, 3700, 400, 3),    # samples that fill a CU's LDS
         ("fp16", "block", 64, 2, 40, 500, 4), ("fp8", "block", 96, 1, 40, 800, 4),
         ("fp32", "auto", 80, 2, 12, 320, 3), ("fp32", "auto", 48, 2, 12, 850, 5), ("fp32", "auto", 192, 1, 12, 200, 9)]


@pytest.mark.parametrize("precision,gridder,N,P,n_ant,n_chan,T", CASES)
def test_two_slots_per_channel_suffice(E, precision, gridder, N, P, n_ant, n_chan, T):
    import torch
    s = dataclasses.replace(box(N, 20, 18, P=P, n_extra=n_ant - 2, seed=6), n_chan=n_chan)
    npp = 4 if P == 2 else 1
    assert 2 * n_chan * npp * N * N * 4 <= E.NOALLOC_MAX_BYTES
    x = torch.from_numpy(np.random.default_rng(3).integers(0, 256, (T, n_chan, n_ant, P), dtype=np.uint8)).cuda()
    a, b = (torch.full((n_chan, npp, N, N), float("nan"), device="cuda") for _ in range(2))
    plan = E.epic_plan([s], precision=precision, gridder=gridder, max_time=T)
    try:
        for n in (T, 2, 1):   # the shorter calls over what the first one left
            E.epic_image_noalloc(plan, [x[:n]], n, [a])
            E.epic_grid_fft_accumulate(plan, [x[:n]], n)
            E.epic_readout(plan, [b], 1)
            torch.cuda.synchronize()
            # the same products of a few spectra, summed in another order
            assert_parity(a.double().cpu().numpy(), b.double().cpu().numpy(), 1e-6, f"{n} spectra")
    finally:
        E.epic_destroy(plan)
