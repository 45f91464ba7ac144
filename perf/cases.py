"""The work that a decoder has this library do, as cases to be timed.

A case is a stretch of constrained diffusion decoding: `steps` consecutive
denoising steps of a batch of partially masked token sequences.  Between two
steps some of the proposed tokens are committed, as in decoding, so that every
step sees sequences that differ from the step before.  `op` says which calls a
pass makes on every step:

* "step":   epic_validate_batch, then epic_select_compatible (the denoising
            step that bench.py measures);
* "decode": the same, then epic_commit_fallback with the step's budget (the
            whole of Alg. 1);
* "first":  epic_lexmemo_build, then epic_validate_batch_noalloc: the first
            check under a grammar that has just been loaded, by a caller that
            has no workspace.

Verdicts and selections are whole numbers, so every output has to be equal.
Witness extraction is not timed here: its bytes are one of many correct
completions and differ from call to call.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_00722_amd import epic
from paper_2606_00722_amd import grammars
from paper_2606_00722_amd import workloads

# vocabulary size and longest token of each language's workload
VOCAB = {"arith": (512, 4), "json": (4096, 6), "smiles": (8192, 4), "clike": (32768, 8)}
BLOCK = 32  # tokens of a block in block decoding ("mask": "block")
BLOCK_MASKED = 0.8  # of the active block, at the first step
BLOCK_REVEALED = 0.2  # of the next block, when one fills
TEXTS = 16  # distinct hidden answers of a batch (each sequence has its own tokens and masks)


def _case(name, lang, B, n, mask, props, steps, op):
    c = {"lang": lang, "B": B, "n": n, "mask": mask, "props": props, "steps": steps, "op": op}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest call: one step over four short expressions
        _case("arith_4x32", "arith", 4, 32, 0.5, 16, 1, "step"),
        # one user's JSON answer, interactive: every call of Alg. 1, odd length
        _case("json_1x97_decode", "json", 1, 97, 0.6, 8, 2, "decode"),
        # the JSON workload: eight answers, half masked
        _case("json_8x128", "json", 8, 128, 0.5, 8, 4, "step"),
        # JSON answers of a serving batch, more checks than compute units
        _case("json_128x128", "json", 128, 128, 0.5, 8, 1, "step"),
        # the SMILES workload
        _case("smiles_16x256", "smiles", 16, 256, 0.6, 8, 2, "step"),
        # the very first step of decoding: nothing committed yet
        _case("smiles_16x256_masked", "smiles", 16, 256, 1.0, 8, 2, "step"),
        # molecules near the end of decoding, odd sizes, with the fallback
        _case("smiles_5x211_decode", "smiles", 5, 211, 0.15, 7, 2, "decode"),
        # the code workload: many tokens per step, masks everywhere
        _case("clike_16x256", "clike", 16, 256, 0.7, 16, 1, "step"),
        # code snippets of a serving batch, more checks than compute units
        _case("clike_48x128", "clike", 48, 128, 0.7, 16, 1, "step"),
        # the code workload at scale, in blocks of 32 tokens
        _case("clike_64x1024_blocks", "clike", 64, 1024, "block", 16, 8, "step"),
        # the same in a smaller, ragged batch, with the fallback
        _case("clike_24x640_blocks_decode", "clike", 24, 640, "block", 16, 4, "decode"),
        # a grammar just loaded: lexing memo of the large vocabulary, first checks
        _case("clike_2x96_first", "clike", 2, 96, 0.8, 8, 1, "first"),
    ]


def _log_int(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    """One more case of the same ranges: any language, batch, length, mask
    ratio and set of calls; the tokens of a batch stay within the listed
    workloads'.  A step has 16 proposals or more, and masks beyond 0.8 come
    with larger batches: a handful of proposals on nothing but masks are all
    valid, whatever they are."""
    lang = rng.choice(["arith", "json", "json", "smiles", "smiles", "clike", "clike", "clike"])
    op = rng.choice(["step", "step", "decode", "first"])
    steps = rng.choice([1, 2, 3])
    props = rng.randint(4, 16)
    mask = round(rng.uniform(0.05, 1.0), 3)
    if lang == "arith":
        n, most = _log_int(rng, 5, 64), 64
    elif lang == "json":
        n = _log_int(rng, 24, 192)
        most = 8192 // n
    elif lang == "smiles":
        n = _log_int(rng, 24, 256)
        most = 4096 // n
    elif rng.random() < 0.5:
        n, mask = _log_int(rng, 65, 1024), "block"
        most = min(64, 32768 // n)
    else:
        n = _log_int(rng, 24, 224)
        most = 2560 // n
    B = max(_log_int(rng, 1, most), -(-16 // props))
    if op == "first":
        B, steps = min(B, 4), 1
    if mask != "block" and B * props < 48:
        mask = min(mask, 0.8)
    return _case(None, lang, B, n, mask, props, steps, op)


def _tokens(rng, text, index, n):
    """`text` as exactly n vocabulary tokens: its single bytes, with as many
    pairs of neighbours joined (into a token of the vocabulary) as are too
    many; None when there are not enough such pairs."""
    parts = [text[i:i + 1] for i in range(len(text))]
    while len(parts) > n:
        order = rng.permutation(len(parts) - 1)
        joined, dead = {}, set()
        for i in order:
            if len(parts) - len(joined) <= n:
                break
            if i in dead or i + 1 in dead or parts[i] + parts[i + 1] not in index:
                continue
            joined[int(i)] = True
            dead.update((int(i), int(i) + 1))
        if not joined:
            return None
        parts = [parts[i] + parts[i + 1] if i in joined else parts[i] for i in range(len(parts)) if i - 1 not in joined]
    ids = [index[p] for p in parts]
    return np.array([a[int(rng.integers(len(a)))] for a in ids], dtype=np.int32)


def _hidden(rng, lang, vocab, B, n):
    """Hidden answers int32 [B, n]: sentences of the grammar, in tokens."""
    index = {}
    for i, s in enumerate(vocab.strings):
        index.setdefault(s, []).append(i)
    out = np.zeros((B, n), dtype=np.int32)
    texts = []
    slack = max(2, n // 16)
    for b in range(B):
        for _ in range(4000):
            if len(texts) < min(B, TEXTS):
                tb = grammars.TextBuilder(lang, rng, extra_space=0.15)
                if not lang.top(tb, n, n + slack):
                    continue
                text = tb.text.encode()
            else:
                text = texts[b % len(texts)]
            row = _tokens(rng, text, index, n) if len(text) >= n else None
            if row is None:
                continue
            if len(texts) < min(B, TEXTS):
                texts.append(text)
            out[b] = row
            break
        else:
            raise RuntimeError("no sentence of %d tokens" % n)
    return out


def _masked(rng, hidden, mask):
    """The sequences of the first step, and the active block of each (block
    decoding) or None."""
    B, n = hidden.shape
    x = hidden.copy()
    if mask == "block":
        nblk = (n + BLOCK - 1) // BLOCK
        active = rng.integers(0, nblk, size=B)
        for b in range(B):
            lo, hi = int(active[b]) * BLOCK, min(n, (int(active[b]) + 1) * BLOCK)
            x[b, hi:] = -1
            x[b, lo + rng.choice(hi - lo, max(1, round(BLOCK_MASKED * (hi - lo))), replace=False)] = -1
        return x, active
    m = min(n, max(1, round(mask * n)))
    for b in range(B):
        x[b, rng.choice(n, m, replace=False)] = -1
    return x, None


def _steps(rng, hidden, mask, props, steps, vocab_size):
    """Per step: the sequences, and the proposals (sequence, position, token,
    confidence).  A proposal is the hidden token half of the time, else any
    token; the hidden ones are committed for the next step."""
    B, n = hidden.shape
    x, active = _masked(rng, hidden, mask)
    out = []
    for _ in range(steps):
        S, P, T, F = [], [], [], []
        nxt = x.copy()
        for b in range(B):
            at = np.flatnonzero(x[b] < 0)
            if active is not None:
                k = int(active[b])
                at = at[(at >= k * BLOCK) & (at < (k + 1) * BLOCK)]
            m = min(props, len(at))
            if m == 0:
                continue
            pos = rng.choice(at, m, replace=False)
            keep = rng.random(m) < 0.5
            S.append(np.full(m, b))
            P.append(pos)
            T.append(np.where(keep, hidden[b, pos], rng.integers(0, vocab_size, size=m)))
            F.append(rng.random(m, dtype=np.float32))
            nxt[b, pos[keep]] = hidden[b, pos[keep]]
            if active is not None and not np.any(nxt[b, k * BLOCK:(k + 1) * BLOCK] < 0) and (k + 1) * BLOCK < n:
                lo, hi = (k + 1) * BLOCK, min(n, (k + 2) * BLOCK)
                active[b] = k + 1
                show = lo + rng.choice(hi - lo, round(BLOCK_REVEALED * (hi - lo)), replace=False)
                nxt[b, show] = hidden[b, show]
        cat = [np.concatenate(a) if a else np.zeros(0) for a in (S, P, T, F)]
        out.append((x, *cat))
        x = nxt
    return out


def prepare(case, seed):
    """What a decoder holds before the pass: the grammar's context with its
    lexing memo, the workspace, and on the device the sequences and proposals
    of every step."""
    rng = np.random.default_rng([int(seed), 2606])
    B, n = case["B"], case["n"]
    size, longest = VOCAB[case["lang"]]
    lang = grammars.language(case["lang"])
    vocab = workloads.make_vocab(rng, lang.alphabet, size, longest)
    steps = _steps(rng, _hidden(rng, lang, vocab, B, n), case["mask"], case["props"], case["steps"], size)
    ctx = epic.Context.from_problem(workloads.arrays(lang, vocab), B, n, B * case["props"])
    ctx.lexmemo_build()
    dev = torch.device("cuda:0")

    def on(a, dt=torch.int32):
        return torch.from_numpy(np.ascontiguousarray(a)).to(dev, dt)

    state = {"op": case["op"], "ctx": ctx, "ws": None if case["op"] == "first" else ctx.alloc_workspace(dev), "steps": []}
    for x, s, p, t, f in steps:
        flags = [torch.zeros(B * case["props"], dtype=torch.uint8, device=dev) for _ in range(3)]  # the batch's most
        budget = np.bincount(s.astype(np.int64), minlength=B)  # all of the step's proposals, as bench.py's fallback
        state["steps"].append({"seqs": on(x), "seq": on(s), "pos": on(p), "tok": on(t), "conf": on(f, torch.float32),
                               "verdict": flags[0], "selected": flags[1], "accepted": flags[2], "budget": on(budget)})
    return state


def run(state):
    ctx, ws, op = state["ctx"], state["ws"], state["op"]
    if op == "first":
        ctx.lexmemo_build()
    out = []
    for d in state["steps"]:
        cand = (d["seqs"], d["seq"], d["pos"], d["tok"])
        if op == "first":
            ctx.validate_noalloc(*cand, d["verdict"])
            out.append({"verdict": d["verdict"]})
            continue
        ctx.validate(*cand, d["verdict"], ws)
        ctx.select(*cand, d["conf"], d["verdict"], d["selected"], ws)
        out.append({"verdict": d["verdict"], "selected": d["selected"]})
        if op == "decode":
            ctx.fallback(*cand, d["conf"], d["verdict"], d["selected"], d["budget"], d["accepted"], ws)
            out[-1]["accepted"] = d["accepted"]
    return out


def work(case):
    """Bytes: every sequence and proposal read once and every flag written
    once, and for "first" the memo table written once (one 16-byte entry per
    token and lexer state).  The path has no floating-point work."""
    B, n, C = case["B"], case["n"], case["B"] * min(case["props"], case["n"])
    step = 4 * B * n + C * (12 + 1)  # sequences, proposals, verdicts
    if case["op"] != "first":
        step += C * (4 + 1)  # confidences, selected
    if case["op"] == "decode":
        step += 4 * B + C  # budgets, accepted
    memo = 0
    if case["op"] == "first":
        size, longest = VOCAB[case["lang"]]
        states = grammars.language(case["lang"]).tables.trans.shape[0]
        memo = size * states * 16 + size * (4 + (longest + 1) // 2) + states * 512
    return {"bytes": case["steps"] * step + memo, "flops": 0}


def tolerance(case):
    return "exact"
