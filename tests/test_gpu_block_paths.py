"""Edges of the kernels that take many tokens or logits at a time: the KV
scatter by whole blocks, the confidence pass over masked logits and the n-gram
scan of one chunk per sequence."""
import numpy as np
import pytest

from paper_2607_03333_amd import synth
from gpu_cases import say
from test_gpu_confidence import THETA, check as check_confidence

pytestmark = pytest.mark.gpu


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
