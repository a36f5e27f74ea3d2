"""The KV write by whole blocks on both sides of its line between workgroups
of one wave and of several per block, and what single tokens, each in a block
of its own, cost on both sides of the line between the scatter by token and
the write by blocks. Exact against the oracle's scatter. And what the write of
long prompts leaves to the step after it."""
import numpy as np
import pytest
import torch

from oracle.kv import scatter_tokens
from paper_2607_03333_amd import spork, synth
from gpu_cases import say
from test_gpu_block_paths import _runs
from test_gpu_kv import _dev, _host, _pools
from test_gpu_logits_rows import _us

pytestmark = pytest.mark.gpu
_DT = {synth.F32: spork.SPORK_DTYPE_F32, synth.BF16: spork.SPORK_DTYPE_BF16}


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bs", [16, 32])
@pytest.mark.parametrize("over", [0, 1])
def test_waves_of_a_block(dtype, d, bs, over):
    hkv, elem = 8, 2 if dtype == synth.BF16 else 4
    waves = min(256, d * bs * elem // 16 * elem // 4) // 64  # of the shared workgroups
    windows = 2048 // waves // hkv
    n = windows * bs - bs + 1 + over  # the most tokens of 2,048 waves, and one more
    rng = np.random.default_rng(n + d)
    lens = [1, bs - 1, bs, bs + 1, 3 * bs + 5, 1, 1]
    lens.append(n - sum(lens))
    nb = sum(x // bs + 2 for x in lens) + 3
    k, v = _pools(rng, dtype, nb, hkv, bs, d)
    dk, dv = _dev(k), _dev(v)
    slots = _runs(rng, nb, bs, lens)
    slots[[5, n - 2]] = -1, nb * bs
    kt, vt = (np.ascontiguousarray(x.reshape(n, hkv, d)) for x in _pools(rng, dtype, n, hkv, 1, d))
    shape = spork.make_shape(hkv, hkv, d, bs, _DT[dtype], 1.0)
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    say(f"  kv write {dtype} d={d} bs={bs} n={n} waves per block {waves}")
    spork.spork_kv_write(shape, dk, dv, nb, torch.from_numpy(slots).cuda(), _dev(kt), _dev(vt), bad)
    torch.cuda.synchronize()
    valid = (slots >= 0) & (slots < nb * bs)
    scatter_tokens(k, v, slots[valid], kt[valid], vt[valid])
    assert int(bad.item()) == 2
    assert np.array_equal(_host(dk, k), k) and np.array_equal(_host(dv, v), v)


@pytest.mark.parametrize("bs", [16, 32])
def test_single_tokens_at_the_line(bs):
    """576 tokens of 8 heads go by blocks, 575 by token: single tokens, the
    worst case of the blocks, cost at most a quarter more there (with one
    wave for a 32-token block it was two fifths)."""
    hkv, d, rng = 8, 128, np.random.default_rng(bs)
    nb = 2000
    shape = spork.make_shape(hkv, hkv, d, bs, spork.SPORK_DTYPE_BF16, 1.0)
    kp = torch.zeros((nb, hkv, bs, d), dtype=torch.bfloat16, device="cuda")
    vp = torch.zeros((nb, hkv, d, bs), dtype=torch.bfloat16, device="cuda")
    slots = torch.from_numpy(_runs(rng, nb, bs, [1] * 576)).cuda()
    x = torch.randn((576, hkv, d), device="cuda").to(torch.bfloat16)
    us = {}
    for n in (575, 576):  # twenty calls in a graph, so that the host does not set the pace
        args = shape, kp, vp, nb, slots[:n], x[:n], x[:n]
        spork.spork_kv_write(*args)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                spork.spork_kv_write(*args)
        us[n] = _us(graph.replay) / 20
    say(f"  us {us}")
    assert us[576] <= 1.25 * us[575]


def test_a_prompts_write_leaves_no_write_back_to_the_next_step():
    """The first decode over freshly written prompts against the same decode
    after a read sweep that evicts whatever the write left in the caches (with
    ordinary stores: up to 256 MB to be written back, a fifth of this step)."""
    hkv, d, bs, n, seqs = 8, 128, 16, 8192, 32  # 1.07 GB of K and V
    nb = seqs * (n // bs + 1)
    cache = spork.spork_cache_create(nb, bs, np.arange(nb))
    try:
        ids = [spork.spork_seq_new(cache) for _ in range(seqs)]
        slots = [torch.from_numpy(spork.spork_seq_append(cache, s, n)[0]).cuda() for s in ids]
        shape = spork.make_shape(8 * hkv, hkv, d, bs, spork.SPORK_DTYPE_BF16, d ** -0.5)
        plan = spork.spork_plan_create(cache, shape, ids, [1] * seqs, list(range(seqs)))
        image = torch.from_numpy(spork.spork_plan_image(plan)).cuda()
        work = torch.empty(spork.spork_plan_get_info(plan)["workspace_bytes"], dtype=torch.uint8, device="cuda")
        spork.spork_workspace_clear(plan, work)
        kp = torch.zeros((nb, hkv, bs, d), dtype=torch.bfloat16, device="cuda")
        vp = torch.zeros((nb, hkv, d, bs), dtype=torch.bfloat16, device="cuda")
        x = torch.randn((n, hkv, d), device="cuda").to(torch.bfloat16)
        q = torch.randn((seqs, 8 * hkv, d), device="cuda").to(torch.bfloat16)
        out, lse = torch.empty_like(q), torch.empty((seqs, 8 * hkv), device="cuda")
        swept = torch.zeros(1 << 28, device="cuda")

        def step(sweep):
            for s in slots:
                spork.spork_kv_write(shape, kp, vp, nb, s, x, x)
            if sweep:
                swept.amax()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            spork.spork_attn_decode(plan, image, q, kp, vp, out, lse, work)
            b.record()
            torch.cuda.synchronize()
            return a.elapsed_time(b) * 1e3

        step(False)
        us = {sweep: float(np.median([step(sweep) for _ in range(9)])) for sweep in (False, True)}
        say(f"  us right after the write {us[False]:.1f}, on swept caches {us[True]:.1f}")
        assert us[False] <= 1.1 * us[True]
    finally:
        spork.spork_plan_destroy(plan)
        spork.spork_cache_destroy(cache)
