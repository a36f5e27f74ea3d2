"""Edges of the kernels that take many tokens or logits at a time: the KV
scatter by whole blocks, the confidence pass over masked logits and the n-gram
scan of one chunk per sequence."""
import numpy as np
import pytest
import torch

import oracle
from oracle.kv import scatter_tokens
from paper_2607_03333_amd import spork, synth
from gpu_cases import say
from test_gpu_confidence import THETA, check as check_confidence
from test_gpu_kv import _dev, _host, _pools
from test_gpu_ngram import check as check_ngram

pytestmark = pytest.mark.gpu


def _runs(rng, nb, bs, lens):
    """Slots of appended runs, each from a random offset of its first block; no slot twice."""
    blocks, out = rng.permutation(nb).tolist(), []
    for n in lens:
        off = int(rng.integers(0, bs))
        own = [blocks.pop() for _ in range((off + n + bs - 1) // bs)]
        out += [own[(off + i) // bs] * bs + (off + i) % bs for i in range(n)]
    return np.array(out, dtype=np.int64)


@pytest.mark.parametrize("dtype,hkv,d,bs", [(synth.F32, 2, 64, 16), (synth.F32, 1, 128, 32), (synth.BF16, 4, 128, 16),
                                            (synth.BF16, 8, 128, 32), (synth.BF16, 3, 64, 16), (synth.F32, 2, 128, 16),
                                            (synth.F32, 2, 64, 32), (synth.BF16, 2, 64, 32)])
@pytest.mark.parametrize("kind", ["below", "least", "one run", "runs", "bad slots", "single tokens"])
def test_kv_write_of_many_tokens_is_exact(dtype, hkv, d, bs, kind):
    least = -(-4608 // hkv)  # tokens of the smallest call that goes by blocks
    lens = {"below": [least - 1], "least": [least], "one run": [least + 277],
            "runs": [least - 400, 1, 15, 16, 17, 31, 32, 33, 333, 2], "bad slots": [least + 50],
            "single tokens": [1] * (least + 6)}[kind]
    bad = (0, 77, least + 49) if kind == "bad slots" else ()
    rng = np.random.default_rng(len(lens) * 100 + d + bs + hkv)
    nb = sum(n // bs + 2 for n in lens) + 3
    k, v = _pools(rng, dtype, nb, hkv, bs, d)
    dk, dv = _dev(k), _dev(v)
    slots = _runs(rng, nb, bs, lens)
    for i, j in enumerate(bad):
        slots[j] = (-1, nb * bs, -(1 << 40))[i]
    kt, vt = (np.ascontiguousarray(x.reshape(len(slots), hkv, d)) for x in _pools(rng, dtype, len(slots), hkv, 1, d))
    shape = spork.make_shape(hkv, hkv, d, bs, spork.SPORK_DTYPE_F32 if dtype == synth.F32 else spork.SPORK_DTYPE_BF16,
                             1.0)
    counter = torch.zeros(1, dtype=torch.int32, device="cuda")
    say(f"  kv write {dtype} hkv={hkv} d={d} bs={bs} n={len(slots)} runs={len(lens)} bad={len(bad)}")
    spork.spork_kv_write(shape, dk, dv, nb, torch.from_numpy(slots).cuda(), _dev(kt), _dev(vt), counter)
    torch.cuda.synchronize()
    valid = (slots >= 0) & (slots < nb * bs)
    scatter_tokens(k, v, slots[valid], kt[valid], vt[valid])
    assert int(counter.item()) == len(bad)
    assert np.array_equal(_host(dk, k), k) and np.array_equal(_host(dv, v), v)


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("vocab", [8, 1024, 4104, 32768, 151936])
@pytest.mark.parametrize("mask", ["lowest", "-inf", "offset"])
def test_confidence_of_masked_and_large_logits(dtype, vocab, mask):
    # Masked to a few tokens (whole threads see only the mask value), or all
    # logits moved by 1500, past the fused form of the exponent's argument.
    b = synth.probe_batch(6, vocab, dtype=dtype, seed=vocab)
    x = b.logits.copy()
    rng = np.random.default_rng(vocab)
    f = np.float32
    if mask == "offset":
        # multiples of 8, which both types hold exactly at this size
        x = (rng.integers(-2, 3, x.shape) * 8 + 1504).astype(f)
    else:
        low = np.frombuffer(np.uint32(0xFF7F0000).tobytes(), dtype=f)[0] if mask == "lowest" else f(-np.inf)
        x = np.full(x.shape, low, dtype=f)
        x[np.arange(len(x)), rng.integers(0, vocab, len(x))] = 3.0
        x[np.arange(len(x)), rng.integers(0, vocab, len(x))] = 2.0
    if dtype == synth.BF16:
        x = (np.ascontiguousarray(x).view(np.uint32) >> 16).astype(np.uint16)
    say(f"confidence {mask} {dtype} V={vocab}")
    check_confidence(x, dtype, b.span_off, THETA, tag=f"{mask} {dtype} V={vocab}")


@pytest.mark.parametrize("n_min,n_max,k", [(1, 1, 1), (1, 32, 50), (3, 8, 300)])
def test_ngram_one_chunk_per_sequence(n_min, n_max, k):
    rng = np.random.default_rng(n_max)
    lens = [0, 1, 2, 31, 32, 33, 34, 255, 256, 257, 1999, 2047, 2048]
    seqs = [rng.integers(0, 2 + i % 3, size=n).astype(np.int32) for i, n in enumerate(lens)]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    check_ngram(np.concatenate(seqs), off, n_min, n_max, k, tag=f"one chunk n {n_min}-{n_max} k {k}")
    # longer than the declared maximum: still scanned whole
    check_ngram(np.tile(seqs[-1], 3), np.array([0, 6144]), n_min, n_max, k, max_len=100, tag="past max_len")
    assert oracle.ngram_propose([seqs[-1]], n_min, n_max, k)[1][0] > 0
