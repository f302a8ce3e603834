"""device_bytes of a dry run: what the real plan allocates, slots apart (their
number follows the workgroups that the card holds)."""
import dataclasses

import pytest

import synth
from coverage_layouts import box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_2301_09662_amd import epic
    return epic


def arrays(kind):
    if kind == "three":
        return [synth.shrink(s, n_chan=2 + k) for k, s in enumerate(synth.workload(4).subs)]
    if kind == "crowded":   # a cell of many antennas pads its slice of the program
        return [dataclasses.replace(box(64, 5, 4, n_extra=300, seed=1), n_chan=3)]
    return [dataclasses.replace(box(64, 20, 18, P=1 if kind == "single" else 2, n_extra=30, seed=1), n_chan=3)]


@pytest.mark.parametrize("kind,precision,gridder,flags", [
    ("dual", "fp32", "auto", ""), ("single", "fp32", "auto", "REMOVE_AUTOCORR"), ("dual", "fp32", "auto", "COMPLEX_WEIGHTS"),
    ("crowded", "fp32", "auto", ""), ("crowded", "fp16", "auto", ""), ("dual", "fp16", "auto", "AUTOTUNE"),
    ("dual", "fp16", "block", ""), ("dual", "fp8", "dense", ""), ("single", "fp16", "direct", ""),
    ("three", "fp16", "auto", "ONE_LAUNCH"), ("three", "fp16", "auto", "")])
def test_dry_run_counts_what_a_plan_allocates(E, kind, precision, gridder, flags):
    subs = arrays(kind)
    got = []
    for dry in (E.EPIC_F_DRY_RUN, 0):
        f = dry | (getattr(E, "EPIC_F_" + flags) if flags else 0)
        plan = E.epic_plan(subs, precision=precision, gridder=gridder, max_time=20, flags=f)
        info = E.epic_plan_query(plan)
        E.epic_destroy(plan)
        slots = sum(info["slots"][k] * s.n_chan * info["npp"][k] * s.grid_n ** 2 * 4 for k, s in enumerate(subs))
        got.append(info["device_bytes"] - slots)
    assert got[0] == got[1]
