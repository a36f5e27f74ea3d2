"""The passes over logits where a row doesn't fill 16-byte vectors: rows that
start and end inside one, rows shorter than one, and what they cost beside
rows that do. A row's first and last elements then go one by one and the rest
by vector, so the maxima are planted at those edges, tied across them, and
the sums of the confidence pass cover every element once (float32 sums
against the oracle's, with test_gpu_confidence's derived tolerance)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_03333_amd import runner, spork, synth
from gpu_cases import run_workload, say
from test_gpu_confidence import LOGPROB_TOL, check as check_confidence

pytestmark = pytest.mark.gpu
_DT = {synth.BF16: spork.SPORK_DTYPE_BF16, synth.F32: spork.SPORK_DTYPE_F32}


def _planted(rows, vocab, rng):
    """Normal logits; row r's maximum at one of the edges, tied with another place in every other row."""
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    at = [0, vocab - 1, vocab // 2, min(vocab - 1, 3), max(0, vocab - 5), min(vocab - 1, 8), max(0, vocab - 9)]
    for r in range(rows):
        x[r, at[r % 7]] = 9.0
        if r % 2:
            x[r, at[(r // 7 + r) % 7]] = 9.0
    return x


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("shift", [0, 1, 7])
@pytest.mark.parametrize("vocab", [1, 2, 3, 5, 7, 8, 9, 13, 16, 17, 31, 511, 1026, 8191, 16387, 33001])
def test_rows_inside_vectors(dtype, vocab, shift):
    rows = 28
    rng = np.random.default_rng(vocab * 8 + shift)
    st = synth.to_storage(_planted(rows, vocab, rng), dtype)
    want = synth.to_f64(st, dtype)
    # `shift` elements into an aligned buffer whose other elements are larger than every logit
    td = torch.bfloat16 if dtype == synth.BF16 else torch.float32
    buf = torch.full((shift + rows * vocab + 16,), 100.0, dtype=td, device="cuda")
    x = buf[shift:shift + rows * vocab].view(rows, vocab)
    x.copy_(runner.to_device(st, dtype, "cuda:0"))
    say(f"rows {dtype} V={vocab} shift={shift}")
    ints = lambda n: torch.full((n,), -7, dtype=torch.int32, device="cuda")  # noqa: E731
    floats = lambda n: torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")  # noqa: E731
    ws = torch.full((max(spork.spork_confidence_workspace_bytes(rows, vocab),
                         spork.spork_verify_workspace_bytes(rows, 0, vocab)) + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    greedy, lp, conf, commit = ints(rows), floats(rows), floats(1), ints(1)
    off = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    spork.spork_probe_confidence(x, _DT[dtype], vocab, rows, off, 1, 0.9, greedy, lp, conf, commit, ws)
    acc, nxt, am = ints(rows), ints(rows), ints(rows)
    spork.spork_verify_accept(None, None, None, None, None, None, None, x, _DT[dtype], vocab, ints(1), rows, 0, acc, nxt,
                              am, ws)
    torch.cuda.synchronize()
    g = oracle.argmax_rows(want)
    assert np.array_equal(greedy.cpu().numpy(), g) and np.array_equal(am.cpu().numpy(), g)
    assert np.array_equal(nxt.cpu().numpy(), g) and not acc.cpu().numpy().any()
    err = np.max(np.abs(lp.cpu().numpy().astype(np.float64) - oracle.top1_logprob(want)))
    assert err <= LOGPROB_TOL, err


@pytest.mark.parametrize("vocab", [2, 6, 333, 8195])
def test_fp32_attention_launch(vocab):
    run_workload(synth.make(0, vocab=vocab), f"fp32 verify V={vocab}").close()


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
def test_first_nan_and_infinity(dtype):
    """Logits are to be finite. What is kept all the same: +inf is the
    maximum, and of a NaN that is a row's first logit the row's index is 0."""
    for vocab in (4096, 4099):
        x = np.random.default_rng(vocab).standard_normal((3, vocab)).astype(np.float32)
        x[0, 777] = np.inf
        x[1, [vocab - 1, 5]] = np.inf
        x[2, 0] = np.nan
        rows = runner.to_device(synth.to_storage(x, dtype), dtype, "cuda:0")
        am = torch.full((3,), -7, dtype=torch.int32, device="cuda")
        z = torch.zeros(3, dtype=torch.int32, device="cuda")
        ws = torch.empty(spork.spork_verify_workspace_bytes(3, 0, vocab) + 256, dtype=torch.uint8, device="cuda")
        spork.spork_verify_accept(None, None, None, None, None, None, None, rows, _DT[dtype], vocab, z, 3, 0, z.clone(),
                                  z.clone(), am, ws)
        torch.cuda.synchronize()
        assert am.cpu().tolist() == [777, 5, 0]


def _us(f, reps=20):
    """Least time of a call among others: what disturbs a measurement only adds to it."""
    best = float("inf")
    f()
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps * 1e3)
    return best


def test_a_vocabulary_that_does_not_fill_vectors_costs_about_the_same():
    """One logit fewer per row, so that most rows start inside a vector: at
    most half as long again (scanned by element it was 2 to 5 times)."""
    times = {}
    for vocab in (151936, 151935):
        x = torch.randn((600, vocab), device="cuda", dtype=torch.bfloat16)
        off = torch.tensor([0, 600], dtype=torch.int32, device="cuda")
        f32 = lambda n: torch.empty(n, device="cuda")  # noqa: E731
        i32 = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")  # noqa: E731
        ws = torch.empty(spork.spork_confidence_workspace_bytes(600, vocab), dtype=torch.uint8, device="cuda")
        out = i32(600), f32(600), f32(1), i32(1)
        conf = _us(lambda: spork.spork_probe_confidence(x, spork.SPORK_DTYPE_BF16, vocab, 600, off, 1, 0.9, *out, ws))
        dw = runner.DeviceWorkload(synth.make(0, vocab=vocab, verify_k=100))
        step = dw.prepare_all()[-1]
        assert step.verify
        times[vocab] = conf, _us(step.run)
        step.dw.close()
    say(f"  us at 151,936 and 151,935: confidence and fp32 verify {times}")
    for aligned, other in zip(times[151936], times[151935]):
        assert other <= 1.5 * aligned


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
@pytest.mark.parametrize("rows,vocab", [(768, 515), (769, 515), (2304, 515), (2305, 515), (2305, 8192), (2305, 16400),
                                        (3583, 16392), (3584, 16392)])
def test_confidence_workgroup_sizes(dtype, rows, vocab):
    """Both sides of every line between 128 and 256 threads: by the number of
    units (768, 2,304, 3,584) and by a unit's length (32 KB)."""
    rng = np.random.default_rng(rows)
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    x[np.arange(rows), rng.integers(0, vocab, rows)] = 7.0
    st = synth.to_storage(x, dtype)
    say(f"confidence {dtype} rows={rows} V={vocab}")
    check_confidence(st, dtype, np.array([0, 5, rows // 2, rows]), tag=f"{dtype} rows={rows} V={vocab}")
