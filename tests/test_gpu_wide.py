"""The 8-wave attention kernels (ranges of more than 8 row tiles), 16-row tiles
for short units and the wide kernel for long ones, where their loops can go
wrong: one to many 32-token stages (a single stage, the first and last
pairs, the ring's depth and one past it), row counts that end inside and on a
32-row tile and on a full slice, both block sizes, and scores that grow along
the context so that the softmax reference moves in every stage. Tolerances
are the parity tests' (bf16 results, gpu_cases)."""
import functools

import numpy as np
import pytest

from paper_2607_03333_amd import runner, synth
from gpu_cases import run_workload

pytestmark = pytest.mark.gpu


def halve_v(wl):
    """V scaled by 1/2 (exact). With a sharp softmax an output is as large as
    single V entries, and three roundings to bf16 (probabilities, partial
    rows, outputs; 2^-9 of max |v| each) bound its error: 3 * 2^-9 * 5 = 0.029
    for standard normal V past the parity tests' 2e-2, 0.015 for half of it."""
    for d in (wl.suffix_v, dict(enumerate(wl.prefix_v))):
        for key, bits in d.items():
            half = synth.f32_to_bf16_bits(0.5 * synth.bf16_bits_to_f32(bits))
            if d is wl.suffix_v:
                wl.suffix_v[key] = half
            else:
                wl.prefix_v[key] = half


@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("k,prefix,gain", [
    (16, 5, 1.0),      # 136 rows, 21 tokens: one stage
    (18, 40, 1.0),     # 152 rows, 58 tokens: two stages
    (19, 77, 4.0),     # 160 rows: five whole tiles, three stages
    (23, 105, 1.0),    # 192 rows, 128 tokens: four whole stages
    (31, 225, 1.0),    # 256 rows: a full slice, 256 tokens: the ring once
    (31, 226, 4.0),    # one token more: nine stages
    (32, 300, 1.0),    # 264 rows: a second slice of 8 rows
    (50, 1000, 12.0),  # 408 rows in two slices, a sharp softmax
])
def test_wide_stage_and_tile_edges(k, prefix, gain, block_size):
    wl = synth.make(3, sessions=2, prefix=prefix, vocab=333, verify_k=k, block_size=block_size, q_gain=gain)
    if gain > 1:
        halve_v(wl)
    dw = run_workload(wl, f"wide K={k} prefix={prefix} bs={block_size}")
    assert dw.steps[0].info["attn_waves"] == 8
    dw.close()


def test_wide_reference_moves_in_every_stage():
    """Keys whose length grows with the position: every stage's scores pass
    the rows' references by more than the slack."""
    wl = synth.make(3, sessions=1, prefix=640, vocab=333, verify_k=16)
    k = synth.bf16_bits_to_f32(wl.prefix_k[0])
    q = synth.bf16_bits_to_f32(wl.steps[0].q)
    k[:] = np.abs(k) * (np.arange(640)[:, None, None] / 64.0).astype(np.float32)
    wl.prefix_k[0] = synth.f32_to_bf16_bits(k)
    wl.steps[0].q = synth.f32_to_bf16_bits(np.abs(q))
    halve_v(wl)
    dw = run_workload(wl, "wide growing scores")
    dw.close()


@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("k,prefix,gain", [
    (24, 1700, 1.0),   # 200 rows: six whole 32-row tiles and 8 rows; 1,725 tokens
    (27, 1764, 4.0),   # 224 rows: seven whole tiles; 1,792 tokens: 56 whole stages
    (31, 1793, 1.0),   # 256 rows, a full slice; 1,825 tokens: an odd number of stages, one token in the last
    (62, 1600, 12.0),  # 504 rows in two slices, a sharp softmax
])
def test_wide_long_units(monkeypatch, k, prefix, gain, block_size):
    """Planned for one compute unit, a unit is a whole range: more than 48
    stages of 13 to 16 row tiles, which the wide kernel runs."""
    monkeypatch.setattr(runner, "DeviceWorkload", functools.partial(runner.DeviceWorkload, n_cu=1))
    wl = synth.make(3, sessions=1, prefix=prefix, vocab=333, verify_k=k, block_size=block_size, q_gain=gain)
    if gain > 1:
        halve_v(wl)
    dw = run_workload(wl, f"wide long K={k} prefix={prefix} bs={block_size}")
    info = dw.steps[0].info
    assert info["attn_waves"] == 8 and info["max_row_tiles"] >= 13
    dw.close()
