"""The 8-wave attention kernels (ranges of more than 8 row tiles) where their
loops can go wrong: one to many 32-token stages (a single stage, the first and
last pairs, the ring's depth and one past it), row counts that end inside and
on a 32-row tile and on a full slice, ranges that start and end inside a
stage, both block sizes, and scores that grow along the context so that the
softmax reference moves in every stage. First the 16-row tiles, which short
and part-filled units run, then the wide kernel, whose plans hold short units
beside long ones. Tolerances are the parity tests' (bf16 results, gpu_cases)."""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2607_03333_amd import runner, spork, synth
from gpu_cases import BF16_RMS, BF16_TOL, LSE_REL, run_workload, say

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


@pytest.mark.parametrize("n_cu", [0, 1])  # cut for a whole chip, and whole ranges as units
@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("k,prefix,gain", [
    (16, 5, 1.0),      # 136 rows, 21 tokens: one stage
    (18, 40, 1.0),     # 152 rows, 58 tokens: two stages
    (19, 77, 4.0),     # 160 rows: five whole tiles; 96 tokens, three whole stages
    (23, 105, 1.0),    # 192 rows, 128 tokens: four whole stages
    (31, 225, 1.0),    # 256 rows: a full slice, 256 tokens: the ring once
    (31, 226, 4.0),    # one token more: nine stages
    (32, 300, 1.0),    # 264 rows: a second slice of 8 rows
    (50, 1000, 12.0),  # 408 rows in two slices, a sharp softmax
])
def test_eight_wave_stage_and_tile_edges(monkeypatch, k, prefix, gain, block_size, n_cu):
    monkeypatch.setattr(runner, "DeviceWorkload", functools.partial(runner.DeviceWorkload, n_cu=n_cu))
    wl = synth.make(3, sessions=2, prefix=prefix, vocab=333, verify_k=k, block_size=block_size, q_gain=gain)
    if gain > 1:
        halve_v(wl)
    dw = run_workload(wl, f"8 waves K={k} prefix={prefix} bs={block_size} n_cu={n_cu}")
    info = dw.steps[0].info
    assert info["attn_waves"] == 8 and info["attn_wide"] == 0
    dw.close()


@pytest.mark.parametrize("n_cu", [0, 1])
def test_eight_wave_reference_moves_in_every_stage(monkeypatch, n_cu):
    """Keys whose length grows with the position: every stage's scores pass
    the rows' references by more than the slack."""
    monkeypatch.setattr(runner, "DeviceWorkload", functools.partial(runner.DeviceWorkload, n_cu=n_cu))
    wl = synth.make(3, sessions=1, prefix=640, vocab=333, verify_k=16)
    k = synth.bf16_bits_to_f32(wl.prefix_k[0])
    q = synth.bf16_bits_to_f32(wl.steps[0].q)
    k[:] = np.abs(k) * (np.arange(640)[:, None, None] / 64.0).astype(np.float32)
    wl.prefix_k[0] = synth.f32_to_bf16_bits(k)
    wl.steps[0].q = synth.f32_to_bf16_bits(np.abs(q))
    halve_v(wl)
    dw = run_workload(wl, f"8 waves growing scores n_cu={n_cu}")
    assert dw.steps[0].info["attn_waves"] == 8 and dw.steps[0].info["attn_wide"] == 0
    dw.close()


@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("k,prefix,gain", [
    (24, 1700, 1.0),   # 200 rows: six whole 32-row tiles and 8 rows; 1,724 tokens
    (27, 1765, 4.0),   # 224 rows: seven whole tiles; 1,792 tokens: 56 whole stages
    (31, 1794, 1.0),   # 256 rows, a full slice; 1,825 tokens: one token in the last stage
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
    assert info["attn_waves"] == 8 and info["attn_wide"] == 1 and info["max_row_tiles"] >= 13
    dw.close()


class _Batch:
    """Threads with random K and V (V halved, see halve_v) in the device pools and on the host."""

    HQ, HKV, D = 8, 1, 128

    def __init__(self, block_size, blocks, growing, seed):
        self.rng, self.blocks, self.growing = np.random.default_rng(seed), blocks, growing
        self.cache = spork.spork_cache_create(blocks, block_size, self.rng.permutation(blocks))
        self.shape = spork.make_shape(self.HQ, self.HKV, self.D, block_size, spork.SPORK_DTYPE_BF16, self.D ** -0.5)
        self.k_pool = torch.full((blocks, self.HKV, block_size, self.D), float("nan"), dtype=torch.bfloat16, device="cuda")
        self.v_pool = torch.full((blocks, self.HKV, self.D, block_size), float("nan"), dtype=torch.bfloat16, device="cuda")
        self.kv = {}  # sequence -> ([K], [V]), float64

    def bf16(self, *shape):
        return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(self.rng.standard_normal(shape).astype(np.float32)))

    def append(self, seq, n):
        slots, cow = spork.spork_seq_append(self.cache, seq, n)
        for src, dst, valid in cow:
            spork.spork_kv_copy(self.shape, self.k_pool, self.v_pool, self.blocks, src, dst, valid)
        k, v = self.bf16(n, self.HKV, self.D), 0.5 * self.bf16(n, self.HKV, self.D)
        if self.growing:
            at = sum(len(x) for x in self.kv[seq][0]) + np.arange(n)
            k = np.abs(k) * (np.minimum(at, 640)[:, None, None] / 64.0).astype(np.float32)
        k, v = synth.f32_to_bf16_bits(k), synth.f32_to_bf16_bits(v)
        spork.spork_kv_write(self.shape, self.k_pool, self.v_pool, self.blocks, torch.from_numpy(slots).cuda(),
                             runner.to_device(k, synth.BF16, "cuda:0"), runner.to_device(v, synth.BF16, "cuda:0"))
        for have, x in zip(self.kv[seq], (k, v)):
            have.append(synth.to_f64(x, synth.BF16))

    def new(self, n):
        seq = spork.spork_seq_new(self.cache)
        self.kv[seq] = ([], [])
        self.append(seq, n)
        return seq

    def fork(self, parent, n):
        seq = spork.spork_fork(self.cache, parent)
        self.kv[seq] = tuple(list(x) for x in self.kv[parent])
        self.append(seq, n)
        return seq

    def plan(self, seqs, rows, groups):
        self.seqs, self.rows = seqs, rows
        self.p = spork.spork_plan_create(self.cache, self.shape, seqs, rows, groups, 1)
        self.info = spork.spork_plan_get_info(self.p)
        host = spork.spork_plan_image(self.p)
        self.image = torch.from_numpy(host).cuda()
        units = host.view(np.int32)[:6 * self.info["n_units"]].reshape(-1, 6)
        self.stages = [int(-(-(hi - lo // 32 * 32) // 32)) for _, lo, hi, _, _, _ in units.tolist()]
        self.starts = [int(lo % 32) for lo in units[:, 1]]
        self.ws = torch.empty(max(256, self.info["workspace_bytes"]), dtype=torch.uint8, device="cuda")

    def run(self, tag):
        n = sum(self.rows)
        q = self.bf16(n, self.HQ, self.D)
        q = synth.f32_to_bf16_bits(np.abs(q) if self.growing else q)
        out = torch.full((n, self.HQ, self.D), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((n, self.HQ), float("nan"), dtype=torch.float32, device="cuda")
        self.ws.fill_(0xFF)
        spork.spork_workspace_clear(self.p, self.ws)
        spork.spork_attn_decode(self.p, self.image, runner.to_device(q, synth.BF16, "cuda:0"), self.k_pool, self.v_pool, out,
                                lse, self.ws)
        torch.cuda.synchronize()
        got, got_lse, row = out.double().cpu().numpy(), lse.double().cpu().numpy(), 0
        worst = err2 = ref2 = 0.0
        for seq, m in zip(self.seqs, self.rows):
            k, v = (np.concatenate(x) for x in self.kv[seq])
            o, ref = oracle.attend(synth.to_f64(q[row:row + m], synth.BF16), k, v, self.shape.sm_scale)
            d = got[row:row + m] - o
            assert np.max(np.abs(got_lse[row:row + m] - ref) / np.maximum(1.0, np.abs(ref))) <= LSE_REL, (tag, seq)
            worst, err2, ref2 = max(worst, float(np.abs(d).max())), err2 + float((d * d).sum()), ref2 + float((o * o).sum())
            row += m
        say(f"  {tag}: {n} rows, max-abs {worst:.2e} rel-rms {(err2 / ref2) ** 0.5:.2e}")
        assert worst <= BF16_TOL and (err2 / ref2) ** 0.5 <= BF16_RMS

    def close(self):
        spork.spork_plan_destroy(self.p)
        spork.spork_cache_destroy(self.cache)


@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("growing", [False, True])
def test_wide_short_units_beside_long_ones(block_size, growing):
    """One wide plan with units of 1 to 10 stages, whole ones and ones that end
    after a single token, 13 to 16 tiles, beside three long ones; a probe of
    30 rows whose private range starts inside a stage. Then the same plan after
    every thread has grown by a token, and by forty more."""
    b = _Batch(block_size, 8000, growing, 7 + block_size)
    seqs, rows, groups = [], [], []

    def thread(seq, n, group):
        seqs.append(seq), rows.append(n), groups.append(group)

    for n in (32, 33, 64, 96, 97, 128, 225, 256, 257, 288, 289, 320):
        thread(b.new(n), 26 + n % 7, -1)
    thread(b.new(13985), 31, -1)  # one token in the last stage
    thread(b.new(14000), 26, -1)
    prompt = b.new(15000)
    probe = b.fork(prompt, 30)
    b.append(prompt, 3)
    thread(prompt, 1, 5), thread(probe, 30, 5)
    b.plan(seqs, rows, groups)
    say(f"wide mix bs={block_size} growing={growing}: units of {sorted(b.stages)} stages")
    assert b.info["attn_waves"] == 8 and b.info["attn_wide"] == 1
    assert {1, 2, 3, 4, 8, 9, 10} <= set(b.stages) and max(b.stages) > 400
    assert block_size == 32 or 16 in b.starts
    b.run("as planned")
    for more in (1, 40):
        for s in seqs:
            b.append(s, more)
        spork.spork_plan_advance(b.p, b.cache, b.image)
        b.run(f"{more} tokens later")
    b.close()
