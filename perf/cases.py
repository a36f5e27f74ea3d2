"""The work that a user of this library has it do, as cases that can be timed.

An attention case is one engine step of one layer: the step's new tokens are
written into the paged pools (``spork_kv_write``), then the batch attends
(``spork_attn_decode``, or ``spork_verify_accept`` when main threads verify
drafts). The other cases are the calls around it: the D2 confidence gate, the
n-gram draft proposer and the KV write of a whole prompt.

``listed()`` are sizes of the library's own workloads and a few that a server
meets beside them; ``draw(rng)`` spreads the same fields over their ranges.
Thread lengths come from the case itself (``lens``), values from the seed.
"""

import math
import random

import numpy as np
import torch

from paper_2607_03333_amd import spork

DEVICE = "cuda:0"
_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_SPORK = {"bf16": spork.SPORK_DTYPE_BF16, "f32": spork.SPORK_DTYPE_F32}
_ELEM = {"bf16": 2, "f32": 4}
PLANTED, CLIP, TIE = 7.0, 6.0, 0.25  # greedy logit, range of the others, chance of a second maximum
THETA = 0.90                         # gate of the confidence call

# Query heads, KV heads and head size of the models the workloads are shaped on.
QWEN3_4B = dict(hq=32, hkv=8, d=128)
QWEN3_32B = dict(hq=64, hkv=8, d=128)
QWEN3_30B_A3B = dict(hq=32, hkv=4, d=128)
SMALL_F32 = dict(hq=4, hkv=2, d=64)


def _attention(name, heads, **kw):
    case = dict(name=name, kind="attention", dtype="bf16", block_size=16, sessions=1, probes=0, prefix_lo=1,
                prefix_hi=1, suffix_lo=1, suffix_hi=1, stagger=0, drafts=0, probe_rows_lo=1, probe_rows_hi=1, vocab=0,
                q_gain=1.0, lens=1)
    case.update(heads)
    case.update(kw)
    return case


def listed():
    return [
        # The smallest call: one session in fp32, the main verifies 4 drafts while its probe decodes.
        _attention("fork-verify-f32", SMALL_F32, dtype="f32", probes=1, prefix_lo=256, prefix_hi=256, suffix_lo=8,
                   suffix_hi=32, drafts=4, vocab=512),
        # One user at a desk: a main thread and one probe, a short context. Latency of the launches.
        _attention("single-session-decode", QWEN3_4B, probes=1, prefix_lo=2000, prefix_hi=2000, suffix_lo=1,
                   suffix_hi=300, q_gain=3.0),
        # A small forked batch (Qwen3-4B heads): 8 mains with a probe each.
        _attention("small-batch-decode", QWEN3_4B, sessions=8, probes=1, prefix_lo=4096, prefix_hi=4096, suffix_lo=1,
                   suffix_hi=2048),
        # Plain decode of unforked sequences of very different lengths, 32-token blocks.
        _attention("ragged-decode-unforked", QWEN3_4B, block_size=32, sessions=96, prefix_lo=3, prefix_hi=8191,
                   q_gain=3.0),
        # A forked decode batch (Qwen3-32B heads): 16 mains with 4 probes each over a 16K prompt.
        _attention("forked-decode", QWEN3_32B, sessions=16, probes=4, prefix_lo=16384, prefix_hi=16384, suffix_lo=1,
                   suffix_hi=2000),
        # The main workload (Qwen3-30B-A3B heads): 64 mains that verify 8 drafts, two probes each that decode.
        _attention("mixed-verify-decode", QWEN3_30B_A3B, sessions=64, probes=2, prefix_lo=32768, prefix_hi=32768,
                   suffix_lo=1, suffix_hi=4096, drafts=8, vocab=151936),
        # The D3 step alone: 16 mains verify 16 drafts.
        _attention("verify-16-drafts", QWEN3_32B, sessions=16, prefix_lo=16383, prefix_hi=16383, drafts=16,
                   vocab=151936),
        # The D3 step with a rejected probe's whole tool call (50 tokens) as drafts.
        _attention("verify-50-drafts", QWEN3_32B, sessions=16, prefix_lo=16383, prefix_hi=16383, drafts=50,
                   vocab=151936, q_gain=3.0),
        # Two probes per session prefill their openers (8 to 50 tokens) over the shared prompt while mains decode.
        _attention("probe-prefill", QWEN3_30B_A3B, sessions=64, probes=2, prefix_lo=32768, prefix_hi=36864,
                   probe_rows_lo=8, probe_rows_hi=50),
        # The D2 gate of 128 probes: tool-name spans of 0 to 16 positions over the whole vocabulary.
        dict(name="probe-confidence", kind="confidence", probes=128, span_hi=16, vocab=151936, dtype="bf16", lens=1),
        # Drafts for 64 agent histories of 32 to 37 thousand tokens.
        dict(name="ngram-drafts", kind="ngram", seqs=64, len_lo=32768, len_hi=36864, n_min=2, n_max=4, k=8, lens=1),
        # The KV of a 15,001-token prompt of one layer goes into its (shuffled) blocks.
        dict(name="prompt-kv-write", kind="kv_write", dtype="bf16", block_size=16, tokens=15001, **{
            k: v for k, v in QWEN3_32B.items() if k != "hq"}),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _draw_attention(rng):
    lens = rng.randrange(1 << 20)
    if rng.random() < 0.15:  # full-precision path: small heads, small batches
        heads, dtype, most = dict(SMALL_F32, d=rng.choice((64, 128))), "f32", 2048
        sessions = _log_int(rng, 1, 4)
    else:
        heads, dtype, most = rng.choice((QWEN3_4B, QWEN3_32B, QWEN3_30B_A3B)), "bf16", 32768
        sessions = _log_int(rng, 1, 64)
    prefix_hi = _log_int(rng, 17, most)
    case = _attention("", heads, dtype=dtype, block_size=rng.choice((16, 16, 32)), sessions=sessions,
                      probes=rng.randint(0, 4), prefix_lo=rng.choice((prefix_hi, 1 + prefix_hi // 2)),
                      prefix_hi=prefix_hi, suffix_hi=_log_int(rng, 1, max(2, most // 8)),
                      q_gain=rng.choice((1.0, 3.0)), lens=lens)
    del case["name"]
    mode = rng.choice(("decode", "verify", "stagger", "prefill"))
    if mode == "verify":
        case["drafts"] = _log_int(rng, 1, 50)
        case["vocab"] = rng.choice((151936, _log_int(rng, 512, 151936)))
    elif mode == "stagger":
        case["stagger"] = _log_int(rng, 5, 400)
        case["probes"] = max(2, case["probes"])
    elif mode == "prefill":
        case["probe_rows_lo"], case["probe_rows_hi"] = 8, _log_int(rng, 8, 50)
        case["probes"] = max(1, case["probes"])
    return case


def draw(rng):
    kind = rng.choice(("attention",) * 7 + ("confidence", "ngram", "kv_write"))
    if kind == "attention":
        while True:
            case = _draw_attention(rng)
            w = work(case)
            most = (4.2e9, 2.0e12) if case["dtype"] == "bf16" else (3e7, 2e9)
            if w["bytes"] <= most[0] and w["flops"] <= most[1]:
                return case
    if kind == "confidence":
        return dict(kind=kind, probes=_log_int(rng, 1, 256), span_hi=rng.randint(2, 16), dtype=rng.choice(("bf16", "f32")),
                    vocab=rng.choice((151936, _log_int(rng, 512, 151936))), lens=rng.randrange(1 << 20))
    if kind == "ngram":
        hi = _log_int(rng, 64, 65536)
        return dict(kind=kind, seqs=_log_int(rng, 1, 128), len_lo=1 + hi // 2, len_hi=hi, n_min=rng.randint(1, 3),
                    n_max=rng.randint(3, 8), k=_log_int(rng, 1, 50), lens=rng.randrange(1 << 20))
    heads = rng.choice((QWEN3_32B, QWEN3_30B_A3B))
    return dict(kind=kind, dtype=rng.choice(("bf16", "bf16", "f32")), block_size=rng.choice((16, 32)),
                tokens=_log_int(rng, 1, 65536), hkv=heads["hkv"], d=heads["d"])


# ---- the batch that an attention case stands for (lengths only) ------------------
def _threads(case):
    """Threads in batch order: (session, is_main, prefix, fork point, own tokens, query rows)."""
    r = random.Random(case["lens"])
    suffix = lambda: _log_int(r, case["suffix_lo"], case["suffix_hi"])  # noqa: E731
    out = []
    for s in range(case["sessions"]):
        prefix = r.randint(case["prefix_lo"], case["prefix_hi"])
        forks = [prefix + (1 + i * case["stagger"] if case["stagger"] else 0) for i in range(case["probes"])]
        last = max(forks + [prefix]) - prefix
        out.append((s, True, prefix, prefix, last + suffix() + case["drafts"], case["drafts"] + 1))
        for f in forks:
            rows = r.randint(case["probe_rows_lo"], case["probe_rows_hi"])
            out.append((s, False, prefix, f, rows if case["probe_rows_hi"] > 1 else suffix(), rows))
    return out


def _span_rows(case):
    r = random.Random(case["lens"])
    return [r.randint(0, case["span_hi"]) for _ in range(case["probes"])]


def _lengths(case):
    r = random.Random(case["lens"])
    return [r.randint(case["len_lo"], case["len_hi"]) for _ in range(case["seqs"])]


def work(case):
    """Each input read once, each output written once; a token of a shared prefix is read once per session."""
    kind = case["kind"]
    if kind == "confidence":
        n = sum(_span_rows(case))
        return {"bytes": n * case["vocab"] * _ELEM[case["dtype"]] + 8 * n + 12 * case["probes"],
                "flops": 3.0 * n * case["vocab"]}
    if kind == "ngram":
        n = sum(_lengths(case))
        return {"bytes": 4 * n + case["seqs"] * (12 + 4 * case["k"]), "flops": 1.0 * n}
    e = _ELEM[case["dtype"]]
    if kind == "kv_write":
        return {"bytes": case["tokens"] * (8 + 4 * case["hkv"] * case["d"] * e), "flops": 0.0}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    tokens = rows = seen = 0
    for _, main, prefix, fork, own, n in _threads(case):
        tokens += own + (prefix if main else 0)  # a probe reads the main's tokens before its fork with the main's own rows
        rows += n
        seen += sum(fork + own - n + r + 1 for r in range(n))
    byt = tokens * 2 * hkv * d * e + 2 * rows * hq * d * e + rows * hq * 4 + rows * 4 * hkv * d * e
    if case["vocab"]:
        byt += case["sessions"] * (case["drafts"] + 1) * (case["vocab"] * e + 8)
    return {"bytes": byt, "flops": 4.0 * seen * hq * d}


def tolerance(case):
    kind = case["kind"]
    if kind in ("ngram", "kv_write"):
        return "exact"
    if kind == "confidence":  # 32-bit sums of exponentials; a gate decision may sit on its threshold
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}  # probabilities and results in bf16


# ---- inputs ----------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(DEVICE).manual_seed(1_000_003 * seed + stream)


def _normal(shape, dtype, gen):
    return torch.randn(shape, dtype=_TORCH[dtype], device=DEVICE, generator=gen)


def _new_kv(case, tokens, seed):
    shape = (tokens, case["hkv"], case["d"])
    return _normal(shape, case["dtype"], _gen(seed, 1)), _normal(shape, case["dtype"], _gen(seed, 2))


def _query(case, rows, seed):
    return _normal((rows, case["hq"], case["d"]), case["dtype"], _gen(seed, 3)) * case["q_gain"]


def _appends(case):
    """The scenario in call order: ("new", t), ("fork", parent, t) and ("append", t, tokens), t = batch index."""
    ops, threads = [], _threads(case)
    t = 0
    while t < len(threads):
        end = t + 1
        while end < len(threads) and not threads[end][1]:
            end += 1
        _, _, prefix, _, own, _ = threads[t]
        ops += [("new", t), ("append", t, prefix)]
        at = prefix
        for p in range(t + 1, end):
            if threads[p][3] > at:
                ops.append(("append", t, threads[p][3] - at))
                at = threads[p][3]
            ops.append(("fork", t, p))
        ops.append(("append", t, prefix + own - at))
        ops += [("append", p, threads[p][4]) for p in range(t + 1, end)]
        t = end
    return threads, [op for op in ops if op[0] != "append" or op[2] > 0]


def _logits(rows, vocab, dtype, seed, rng):
    """Clipped normal logits with a planted maximum per row (a tie now and then); (logits, greedy token per row)."""
    x = torch.randn((rows, vocab), dtype=_TORCH[dtype], device=DEVICE, generator=_gen(seed, 4)).clamp_(-CLIP, CLIP)
    target = rng.integers(0, vocab, rows)
    partner = np.where(rng.random(rows) < TIE, (target + 1 + rng.integers(0, vocab - 1, rows)) % vocab, target)
    r = torch.arange(rows, device=DEVICE)
    for t in (target, partner):
        x[r, torch.from_numpy(t).to(DEVICE)] = PLANTED
    return x, np.minimum(target, partner)


class _Handles:
    """The block manager and plan of a state, destroyed with it."""

    def __init__(self, cache, plan=None):
        self.cache, self.plan = cache, plan

    def __del__(self):
        if self.plan is not None:
            spork.spork_plan_destroy(self.plan)
        spork.spork_cache_destroy(self.cache)


def _prepare_attention(case, seed):
    threads, ops = _appends(case)
    bs, dtype, hkv, d = case["block_size"], case["dtype"], case["hkv"], case["d"]
    blocks = 8 + sum(op[2] // bs + 2 for op in ops if op[0] == "append")
    rng = np.random.default_rng(seed)
    cache = spork.spork_cache_create(blocks, bs, rng.permutation(blocks))
    handles = _Handles(cache)
    shape = spork.make_shape(case["hq"], hkv, d, bs, _SPORK[dtype], 1.0 / math.sqrt(d))
    k_pool = torch.zeros((blocks, hkv, bs, d), dtype=_TORCH[dtype], device=DEVICE)
    v_pool = torch.zeros((blocks, hkv, d, bs), dtype=_TORCH[dtype], device=DEVICE)
    k, v = _new_kv(case, sum(op[2] for op in ops if op[0] == "append"), seed)
    seq, at, step = {}, 0, {}
    for op in ops:
        if op[0] == "new":
            seq[op[1]] = spork.spork_seq_new(cache)
        elif op[0] == "fork":
            seq[op[2]] = spork.spork_fork(cache, seq[op[1]])
        else:
            t, n = op[1:]
            slots, cow = spork.spork_seq_append(cache, seq[t], n)
            for src, dst, valid in cow:
                spork.spork_kv_copy(shape, k_pool, v_pool, blocks, src, dst, valid)
            spork.spork_kv_write(shape, k_pool, v_pool, blocks, torch.from_numpy(slots).to(DEVICE), k[at:at + n],
                                 v[at:at + n])
            step.setdefault(t, []).extend(zip(slots.tolist()[-64:], range(at, at + n)[-64:]))
            at += n
    rows = [th[5] for th in threads]
    new = [x for t, n in enumerate(rows) for x in step[t][-n:]]  # the tokens that this step adds
    idx = torch.tensor([i for _, i in new], device=DEVICE)
    plan = spork.spork_plan_create(cache, shape, [seq[t] for t in range(len(threads))], rows, [th[0] for th in threads])
    handles.plan = plan
    n_rows = sum(rows)
    st = dict(kind="attention", handles=handles, plan=plan, shape=shape, blocks=blocks, k_pool=k_pool, v_pool=v_pool,
              slots=torch.tensor([s for s, _ in new], device=DEVICE), k_new=k[idx].contiguous(),
              v_new=v[idx].contiguous(), image=torch.from_numpy(spork.spork_plan_image(plan)).to(DEVICE),
              q=_query(case, n_rows, seed),
              out=torch.empty((n_rows, case["hq"], d), dtype=_TORCH[dtype], device=DEVICE),
              lse=torch.empty((n_rows, case["hq"]), dtype=torch.float32, device=DEVICE), vocab=case["vocab"])
    ws = (spork.spork_plan_get_info(plan)["workspace_bytes"] + 255) // 256 * 256
    if case["vocab"]:
        n, kd, vocab = case["sessions"], case["drafts"], case["vocab"]
        logits, greedy = _logits(n * (kd + 1), vocab, dtype, seed, rng)
        match = np.minimum(rng.geometric(0.3, n) - 1, kd)
        greedy = greedy.reshape(n, kd + 1)[:, :kd]
        wrong = (greedy + 1 + rng.integers(0, vocab - 1, greedy.shape)) % vocab
        drafts = np.where(np.arange(kd)[None] < match[:, None], greedy, wrong).astype(np.int32)
        ints = lambda m: torch.zeros(m, dtype=torch.int32, device=DEVICE)  # noqa: E731
        st.update(logits=logits, ltype=_SPORK[dtype], drafts=torch.from_numpy(drafts).to(DEVICE), n=n, kd=kd,
                  accept_len=ints(n), next_token=ints(n), argmax=ints(n * (kd + 1)))
        ws += spork.spork_verify_workspace_bytes(n, kd, vocab)
    st["workspace"] = torch.empty(max(ws, 256), dtype=torch.uint8, device=DEVICE)
    spork.spork_workspace_clear(plan, st["workspace"])
    return st


def _probe_logits(case, rows, seed):
    """Normal logits, one token of a row boosted so that its probability spreads over (0.02, 1)."""
    x = _normal((rows, case["vocab"]), case["dtype"], _gen(seed, 5))
    rng = np.random.default_rng(seed)
    boost = math.log(case["vocab"]) + 0.5 + rng.uniform(-4, 8, rows)
    r, c = torch.arange(rows, device=DEVICE), torch.from_numpy(rng.integers(0, case["vocab"], rows)).to(DEVICE)
    x[r, c] += torch.from_numpy(boost).to(DEVICE).to(x.dtype)
    return x


def _histories(case, seed):
    """Agent histories: segments (mean 16 tokens) of fresh Zipf-ranked tokens, a third of them copies of earlier spans."""
    rng = np.random.default_rng(seed)
    seqs = []
    for n in _lengths(case):
        t = ((rng.zipf(1.2, n) - 1) % 151936).astype(np.int32)
        cuts = np.cumsum(rng.geometric(1 / 16, n // 16 + 2))
        copies, where = rng.random(len(cuts)) < 0.35, rng.random(len(cuts))
        for a, b, c, w in zip(cuts[:-1].tolist(), cuts[1:].tolist(), copies.tolist(), where.tolist()):
            b = min(b, n)
            if c and b > a:
                src = int(w * max(1, a - (b - a)))
                t[a:b] = t[src:src + b - a].copy()
        seqs.append(t)
    return np.concatenate(seqs), np.cumsum([0] + [len(s) for s in seqs]).astype(np.int64)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "attention":
        return _prepare_attention(case, seed)
    ints = lambda *m: torch.zeros(m, dtype=torch.int32, device=DEVICE)  # noqa: E731
    floats = lambda m: torch.zeros(m, dtype=torch.float32, device=DEVICE)  # noqa: E731
    if kind == "confidence":
        off = np.cumsum([0] + _span_rows(case)).astype(np.int32)
        rows, n = int(off[-1]), case["probes"]
        ws = spork.spork_confidence_workspace_bytes(rows, case["vocab"])
        return dict(kind=kind, logits=_probe_logits(case, rows, seed), ltype=_SPORK[case["dtype"]], vocab=case["vocab"],
                    rows=rows, off=torch.from_numpy(off).to(DEVICE), n=n, argmax=ints(rows), logprob=floats(rows),
                    confidence=floats(n), commit=ints(n),
                    workspace=torch.empty(max(ws, 256), dtype=torch.uint8, device=DEVICE))
    if kind == "ngram":
        tokens, off = _histories(case, seed)
        n, most = case["seqs"], max(_lengths(case))
        ws = spork.spork_ngram_workspace_bytes(n, most)
        return dict(kind=kind, tokens=torch.from_numpy(tokens).to(DEVICE), off=torch.from_numpy(off).to(DEVICE), n=n,
                    most=most, n_min=case["n_min"], n_max=case["n_max"], k=case["k"], drafts=ints(n, case["k"]),
                    n_drafts=ints(n), workspace=torch.empty(max(ws, 256), dtype=torch.uint8, device=DEVICE))
    bs, hkv, d, n = case["block_size"], case["hkv"], case["d"], case["tokens"]
    blocks = n // bs + 9
    cache = spork.spork_cache_create(blocks, bs, np.random.default_rng(seed).permutation(blocks))
    handles = _Handles(cache)
    slots, _ = spork.spork_seq_append(cache, spork.spork_seq_new(cache), n)
    k, v = _new_kv(case, n, seed)
    zeros = lambda *m: torch.zeros(m, dtype=_TORCH[case["dtype"]], device=DEVICE)  # noqa: E731
    return dict(kind=kind, handles=handles, blocks=blocks, slots=torch.from_numpy(slots).to(DEVICE), k_new=k, v_new=v,
                shape=spork.make_shape(hkv, hkv, d, bs, _SPORK[case["dtype"]], 1.0 / math.sqrt(d)),
                k_pool=zeros(blocks, hkv, bs, d), v_pool=zeros(blocks, hkv, d, bs))


# ---- one pass ----------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "confidence":
        spork.spork_probe_confidence(s["logits"], s["ltype"], s["vocab"], s["rows"], s["off"], s["n"], THETA,
                                     s["argmax"], s["logprob"], s["confidence"], s["commit"], s["workspace"])
        return {k: s[k] for k in ("argmax", "logprob", "confidence", "commit")}
    if kind == "ngram":
        spork.spork_ngram_propose(s["tokens"], s["off"], s["n"], s["most"], s["n_min"], s["n_max"], s["k"], s["drafts"],
                                  s["n_drafts"], s["workspace"])
        return {k: s[k] for k in ("drafts", "n_drafts")}
    spork.spork_kv_write(s["shape"], s["k_pool"], s["v_pool"], s["blocks"], s["slots"], s["k_new"], s["v_new"])
    if kind == "kv_write":
        return {k: s[k] for k in ("k_pool", "v_pool")}
    if not s["vocab"]:
        spork.spork_attn_decode(s["plan"], s["image"], s["q"], s["k_pool"], s["v_pool"], s["out"], s["lse"],
                                s["workspace"])
        return {k: s[k] for k in ("out", "lse")}
    spork.spork_verify_accept(s["plan"], s["image"], s["q"], s["k_pool"], s["v_pool"], s["out"], s["lse"], s["logits"],
                              s["ltype"], s["vocab"], s["drafts"], s["n"], s["kd"], s["accept_len"], s["next_token"],
                              s["argmax"], s["workspace"])
    return {k: s[k] for k in ("out", "lse", "accept_len", "next_token", "argmax")}


# ---- the same in 64 bits, by plain torch --------------------------------------------
def _exact_attention(case, seed):
    threads, ops = _appends(case)
    k, v = _new_kv(case, sum(op[2] for op in ops if op[0] == "append"), seed)
    q = _query(case, sum(th[5] for th in threads), seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    runs, at = {}, 0  # thread -> token runs (first, count) of its context
    for op in ops:
        if op[0] == "new":
            runs[op[1]] = []
        elif op[0] == "fork":
            runs[op[2]] = list(runs[op[1]])
        else:
            runs[op[1]].append((at, op[2]))
            at += op[2]
    outs, lses, row = [], [], 0
    for t, th in enumerate(threads):
        n = th[5]
        kk, vv = (torch.cat([x[a:a + m] for a, m in runs[t]]).double().permute(1, 2, 0).contiguous() for x in (k, v))
        qq = q[row:row + n].double().reshape(n, hkv, hq // hkv, d).permute(1, 0, 2, 3).reshape(hkv, -1, d).contiguous()
        s = torch.bmm(qq, kk) / math.sqrt(d)  # [hkv, n * heads, context]
        length = kk.shape[2]
        last = length - n + torch.arange(n, device=DEVICE).repeat_interleave(hq // hkv)
        s.masked_fill_(torch.arange(length, device=DEVICE)[None] > last[:, None], -math.inf)
        lse = torch.logsumexp(s, 2)
        o = torch.bmm(torch.exp_(s.sub_(lse[..., None])), vv.permute(0, 2, 1).contiguous())
        outs.append(o.reshape(hkv, n, hq // hkv, d).permute(1, 0, 2, 3).reshape(n, hq, d))
        lses.append(lse.reshape(hkv, n, hq // hkv).permute(1, 0, 2).reshape(n, hq))
        row += n
    got = {"out": torch.cat(outs), "lse": torch.cat(lses)}
    if case["vocab"]:
        got.update(accept_len=None, next_token=None, argmax=None)
    return got


def exact(case, seed):
    if case["kind"] == "attention":
        return _exact_attention(case, seed)
    if case["kind"] != "confidence":
        return None
    spans = _span_rows(case)
    x = _probe_logits(case, sum(spans), seed)
    lp = torch.cat([r.double().log_softmax(1).amax(1) for r in x.split(64)] + [torch.zeros(0, device=DEVICE).double()])
    conf = [r[1:].min().exp() if len(r) > 1 else torch.ones((), device=DEVICE).double() for r in lp.split(spans)]
    return {"argmax": None, "logprob": lp, "confidence": torch.stack(conf), "commit": None}
