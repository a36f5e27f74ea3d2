"""Softmax scales of zero and below, which the planner accepts like any finite
one: the causal rule's masked positions stay out whatever the scale's sign.
Every attention kernel against the oracle (tolerances of the parity tests),
with verify rows (causal) and ranges that start and end inside a stage."""
import functools

import pytest

from paper_2607_03333_amd import runner, synth
from gpu_cases import run_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [0.0, -0.0, -0.08838834764])
@pytest.mark.parametrize("kernel,make", [
    ("fp32", lambda: synth.make(0)),
    ("4 waves", lambda: synth.make(4, sessions=2, prefix=333, vocab=333)),
    ("8 waves", lambda: synth.make(3, sessions=2, prefix=105, vocab=333, verify_k=23)),
    ("8 waves, 32-token blocks", lambda: synth.make(3, sessions=2, prefix=105, vocab=333, verify_k=23, block_size=32)),
    ("wide", lambda: synth.make(3, sessions=1, prefix=1700, vocab=333, verify_k=24)),
    ("wide, 32-token blocks", lambda: synth.make(3, sessions=1, prefix=1700, vocab=333, verify_k=24, block_size=32)),
])
def test_scales_up_to_zero(monkeypatch, kernel, make, scale):
    if "wide" in kernel:  # planned for one compute unit: units long enough for the wide kernel
        monkeypatch.setattr(runner, "DeviceWorkload", functools.partial(runner.DeviceWorkload, n_cu=1))
    wl = make()
    wl.sm_scale = scale
    dw = run_workload(wl, f"{kernel} scale {scale}")
    info = dw.steps[-1].info
    assert info["attn_waves"] == {"f": 1, "4": 4}.get(kernel[0], 8) and info["attn_wide"] == int("wide" in kernel)
    dw.close()
