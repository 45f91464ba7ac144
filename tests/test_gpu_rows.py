"""Chart rows at the edges of the walk's passes, on the device through the C
ABI, against the oracle's verdicts and selections (whole numbers, so equal):
rows with more entries than a wavefront takes at a time, more slots than
wavefronts share out at once, many in-edges, runs of more tokens than one
wavefront scans, calls with more candidates than CUs, whose selection resumes
from base walks, masked runs of one and of eight class nodes, and buffers that
overflow."""
import numpy as np
import pytest

from paper_2606_00722_amd import grammars as G
from paper_2606_00722_amd import lexspec as lx
from paper_2606_00722_amd import workloads as W

pytestmark = pytest.mark.gpu

NTH = 8


@pytest.fixture(scope="module")
def gpu_mod():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to the gpu-marked tests")
    from tests import gpu_util

    return gpu_util


def masked_case(preset, B, n, pattern, seed):
    """Hidden answers of the preset with masks at a fixed pattern, proposals
    at masked positions (the hidden token half of the time)."""
    inst = W.make_instance(preset, seed, B=B, n=n)
    x = inst.hidden.copy()
    if pattern == "alternate":  # as many masked runs, and slots in their rows, as fit
        x[:, 1::2] = W.MASK
    elif pattern == "third":
        x[:, ::3] = W.MASK
    elif pattern == "long run":  # over 64 fixed tokens between two masked runs
        x[:, :2] = W.MASK
        x[:, -2:] = W.MASK
    elif pattern == "one run":
        x[:, n // 4:3 * n // 4] = W.MASK
    return inst, x.astype(np.int32)


def proposals(inst, x, props, rng):
    seq, pos, tok = [], [], []
    for b in range(x.shape[0]):
        at = np.flatnonzero(x[b] == W.MASK)
        p = rng.choice(at, min(props, len(at)), replace=False)
        keep = rng.random(len(p)) < 0.5
        seq.append(np.full(len(p), b))
        pos.append(p)
        tok.append(np.where(keep, inst.hidden[b, p], rng.integers(0, inst.vocab.size, len(p))))
    seq, pos, tok = (np.concatenate(a).astype(np.int32) for a in (seq, pos, tok))
    return seq, pos, tok, rng.random(len(seq), dtype=np.float32)


@pytest.mark.parametrize("preset,B,n,pattern,props", [
    (1, 3, 129, "alternate", 8),    # one word a set, 64 masked runs
    (1, 2, 200, "long run", 4),     # a run of 196 tokens
    (2, 2, 128, "alternate", 6),    # four words
    (2, 2, 90, "long run", 4),
    (3, 2, 97, "third", 6),         # one class node a run
    (4, 2, 64, "alternate", 6),     # sixteen words
    (4, 2, 96, "long run", 4),
    (4, 2, 63, "one run", 6),
    (2, 40, 32, "third", 8),        # 320 candidates, more than CUs: selection from base walks
    (4, 24, 24, "third", 8),        # 192 candidates and 48 base walks: they fit on the CUs
    (4, 33, 24, "third", 8),        # 264 candidates: more than CUs
    (4, 31, 24, "third", 8),        # 248 candidates, but not with 62 base walks: no sharing
])
def test_rows_at_pass_edges(preset, B, n, pattern, props, gpu_mod, oracle_lib):
    rng = np.random.default_rng([preset, B, n])
    inst, x = masked_case(preset, B, n, pattern, 7)
    seq, pos, tok, conf = proposals(inst, x, props, rng)
    p = oracle_lib.problem_from(inst.lang, inst.vocab)
    g = gpu_mod.Gpu(W.arrays(inst.lang, inst.vocab), B, n, len(seq))
    want = oracle_lib.validate_batch(p, x, seq, pos, tok, NTH)
    for _ in range(3):  # the order in which wavefronts add to a row differs from call to call
        assert np.array_equal(g.validate(x, seq, pos, tok), want)
    assert g.errors() == 0
    want_s, counts, st = oracle_lib.select(p, x, seq, pos, tok, conf, want, NTH)
    sel, got_counts = g.select(x, seq, pos, tok, conf, want)
    assert st == 0 and g.errors() == 0
    assert np.array_equal(sel, want_s) and tuple(got_counts) == tuple(int(c) for c in counts)


@pytest.mark.parametrize("B,props,graphs", [
    (300, 1, 1),  # one candidate a sequence: Alg. 4 makes no check, no cover walk is made for it
    (129, 2, 2),  # 258 candidates, more than CUs: validation walks the cover graphs' base walks too
    (128, 2, 0),  # 256: each has a CU, and base walks would not fit beside them
])
def test_base_walks_of_wide_calls(B, props, graphs, gpu_mod, oracle_lib):
    """How many graphs of a sequence validation walks for prefix sharing."""
    import torch

    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the calls are sized for 256 CUs")
    inst, x = masked_case(1, B, 12, "third", 5)
    seq, pos, tok, conf = proposals(inst, x, props, np.random.default_rng(3))
    assert len(seq) == B * props
    p = oracle_lib.problem_from(inst.lang, inst.vocab)
    g = gpu_mod.Gpu(W.arrays(inst.lang, inst.vocab), B, x.shape[1], len(seq))
    want = oracle_lib.validate_batch(p, x, seq, pos, tok, NTH)
    assert np.array_equal(g.validate(x, seq, pos, tok), want)
    assert g.ctx.kernel_stats()["base"]["work"][0] == B * graphs
    want_s, _, st = oracle_lib.select(p, x, seq, pos, tok, conf, want, NTH)
    sel, _ = g.select(x, seq, pos, tok, conf, want)
    assert st == 0 and g.errors() == 0 and np.array_equal(sel, want_s)


@pytest.mark.parametrize("name", ["tiny_paren", "tiny_expr", "tiny_ab"])
def test_long_rows_of_tiny_languages(name, gpu_mod, oracle_lib):
    """Nullable productions and a three-class lexer (completion by iteration)
    with every other token masked: the verdicts of 40 masked positions, a token
    each, equal the oracle's."""
    from tests.util import custom_vocab

    lang = G.language(name)
    vocab = custom_vocab(lang, {"tiny_paren": ["((", "))", "()"], "tiny_expr": ["a+", "(a", " a"],
                                "tiny_ab": ["ab", "ba", "cc"]}[name])
    rng = np.random.default_rng(11)
    n = 33
    x = rng.integers(0, vocab.size, size=(6, n)).astype(np.int32)
    x[:, ::2] = W.MASK
    x[0, 1::4] = W.MASK
    x[1] = W.MASK
    at = np.argwhere(x == W.MASK)
    at = at[rng.choice(len(at), 40, replace=False)]
    seq, pos = at[:, 0].astype(np.int32), at[:, 1].astype(np.int32)
    tok = rng.integers(0, vocab.size, size=len(at)).astype(np.int32)
    p = oracle_lib.problem_from(lang, vocab)
    g = gpu_mod.Gpu(W.arrays(lang, vocab), x.shape[0], n, len(at))
    assert np.array_equal(g.validate(x, seq, pos, tok), oracle_lib.validate_batch(p, x, seq, pos, tok, NTH))
    assert g.errors() == 0


def test_one_gap_class_at_sixteen_words(gpu_mod, oracle_lib):
    """The SMILES-like grammar, one class node a masked run, padded to sixteen
    words a set."""
    from tests.util import pad_language

    inst, x = masked_case(3, 3, 50, "third", 9)
    lang = pad_language(inst.lang)
    seq, pos, tok, conf = proposals(inst, x, 8, np.random.default_rng(2))
    p = oracle_lib.problem_from(lang, inst.vocab)
    g = gpu_mod.Gpu(W.arrays(lang, inst.vocab), 3, 50, len(seq))
    assert (g.ctx.gap_classes, g.ctx.item_words) == (1, 16)
    want = oracle_lib.validate_batch(p, x, seq, pos, tok, NTH)
    assert np.array_equal(g.validate(x, seq, pos, tok), want)
    want_s, counts, st = oracle_lib.select(p, x, seq, pos, tok, conf, want, NTH)
    sel, got_counts = g.select(x, seq, pos, tok, conf, want)
    assert st == 0 and g.errors() == 0
    assert np.array_equal(sel, want_s) and tuple(got_counts) == tuple(int(c) for c in counts)


def pairs_language(only_z=False):
    """Six pairs of letters x, y where x then y always lexes as xy, so that no
    lexeme y follows a lexeme x: a lexer with eight gap classes.  Runs of z are
    one lexeme, so that a lexeme can span any number of masked runs.  S is
    right-recursive: a sequence of any lexemes, which completes at every origin
    before when it completes, or z runs with a between them."""
    firsts, seconds = "acegik", "bdfhjl"
    pats = [w for x, y in zip(firsts, seconds) for w in (x, x + y, y)]
    names = ["T%d" % i for i in range(len(pats))] + ["Z"]
    prods = [("S", (t, "S")) for t in names] + [("S", (names[0],)), ("S", ("Z", "Z", "S"))]
    if only_z:
        prods = [("S", ("Z", names[0], "S")), ("S", ("Z",))]
    g = G.Grammar(names, ["S"], prods, "S")
    rules = [lx.LexerRule(n, lx.lit(w), g.tid[n]) for n, w in zip(names, pats)]
    rules.append(lx.LexerRule("Z", lx.plus(lx.cls("z")), g.tid["Z"]))
    return G.Language("pairs", g, rules, firsts + seconds + "z", {}, wordish=frozenset())


def masked_runs(idx, runs, between, n, fill):
    """`runs` masked tokens with the token `between` after each, then `fill`."""
    x = np.full(n, idx[fill], np.int32)
    x[0:2 * runs:2] = W.MASK
    x[1:2 * runs:2] = idx[between]
    return x


@pytest.mark.parametrize("only_z,pad,words", [(False, 0, 4), (False, 2, 16), (True, 0, 1)])
def test_many_gap_classes(only_z, pad, words, gpu_mod, oracle_lib):
    """Eight class nodes a masked run: completion by iteration, at 4 and 16
    words a set; and lexemes in progress over up to 18 masked runs, each of
    which adds two, whose frontier entries enter the last runs by more than 256
    label sets."""
    from tests.util import custom_vocab, pad_language

    lang = pairs_language(only_z)
    vocab = custom_vocab(lang, ["ab", "zz", "ca"])
    for _ in range(pad):
        lang = pad_language(lang)
    idx = {s: i for i, s in enumerate(vocab.strings)}
    rng = np.random.default_rng(17)
    n, runs = (38, 18) if only_z else (14, 5)
    rows = [masked_runs(idx, runs, b"z", n, b"a"), masked_runs(idx, runs, b"z", n, b"zz"),
            masked_runs(idx, 4, b"c", n, b"a")]
    for _ in range(5):
        x = np.full(n, idx[b"z"], np.int32) if only_z else rng.integers(0, vocab.size, n).astype(np.int32)
        x[rng.choice(n, 6, replace=False)] = W.MASK
        rows.append(x)
    rows.append(np.full(n, W.MASK, np.int32))
    x = np.stack(rows)
    at = np.argwhere(x == W.MASK)
    seq, pos = np.repeat(at, 3, axis=0).astype(np.int32).T
    tok = rng.integers(0, vocab.size, size=len(seq)).astype(np.int32)
    p = oracle_lib.problem_from(lang, vocab)
    g = gpu_mod.Gpu(W.arrays(lang, vocab), len(x), n, len(seq))
    assert (g.ctx.gap_classes, g.ctx.item_words) == (8, words)
    want = oracle_lib.validate_batch(p, x, seq, pos, tok, NTH)
    got = g.validate(x, seq, pos, tok)
    assert g.errors() == 0
    assert np.array_equal(got, want) and 0 < int(want.sum()) < len(want)
    one = np.unique(at[:, 0] * n + at[:, 1], return_index=True)[1] * 3  # a candidate a position
    s1, p1, t1 = seq[one], pos[one], tok[one]
    conf = rng.random(len(one), dtype=np.float32)
    want_s, counts, st = oracle_lib.select(p, x, s1, p1, t1, conf, want[one], NTH)
    sel, got_counts = g.select(x, s1, p1, t1, conf, want[one])
    assert st == 0 and g.errors() == 0
    assert np.array_equal(sel, want_s) and tuple(got_counts) == tuple(int(c) for c in counts)


# the error word's bits for the buffer that overflowed; ENTRIES also stands for
# any buffer of the base walk that a walk would have resumed from
SLOTS, ENTRIES, FRONTIER = 1 << 9, 1 << 12, 1 << 15


@pytest.mark.parametrize("runs,between,only_z,buffer", [(30, b"a", False, SLOTS), (56, b"z", True, FRONTIER)])
def test_buffers_that_overflow(runs, between, only_z, buffer, gpu_mod, oracle_lib):
    """Sequences whose rows have more origins than slots, or whose lexeme in
    progress has more frontier entries than fit: verdict 2 and
    EPIC_DEV_CAPACITY, and the walks that a workgroup makes after such a one
    (more candidates than chart slots) agree with the oracle, as do the
    selections of the other sequences."""
    from paper_2606_00722_amd import epic
    from tests.util import custom_vocab

    lang = pairs_language(only_z)
    vocab = custom_vocab(lang, ["ab", "zz", "ca"])
    idx = {s: i for i, s in enumerate(vocab.strings)}
    n = 116
    full = masked_runs(idx, runs, between, n, between)
    rng = np.random.default_rng(23)
    some = np.full((3, n), idx[between], np.int32)
    some[1] = rng.integers(0, vocab.size, n)
    for b in range(3):
        some[b, rng.choice(n, 4, replace=False)] = W.MASK
    x = np.concatenate([full[None], some])
    at = np.argwhere(some == W.MASK)
    half = 1024  # as many walks as run at once at most: every workgroup meets the overflow first
    seq = np.concatenate([np.zeros(half), 1 + np.resize(at[:, 0], half)]).astype(np.int32)
    pos = np.concatenate([np.full(half, 2 * (runs - 1)), np.resize(at[:, 1], half)]).astype(np.int32)
    tok = np.concatenate([np.full(half, idx[between]), rng.integers(0, vocab.size, half)]).astype(np.int32)
    p = oracle_lib.problem_from(lang, vocab)
    want = oracle_lib.validate_batch(p, x, seq[half:], pos[half:], tok[half:], NTH)
    assert 0 < int(want.sum()) < half
    g = gpu_mod.Gpu(W.arrays(lang, vocab), len(x), n, 2 * half)
    out = g.torch.full((2 * half,), 7, dtype=g.torch.uint8, device=g.dev)
    g.ctx.validate_noalloc(g.t(x), g.t(seq), g.t(pos), g.t(tok), out)
    g.torch.cuda.synchronize()
    assert g.errors() == epic.DEV_CAPACITY | buffer
    for got in (out.cpu().numpy(), g.validate(x, seq, pos, tok)):
        assert np.all(got[:half] == 2) and np.array_equal(got[half:], want)
    assert g.errors() & ~(buffer | ENTRIES) == epic.DEV_CAPACITY
    # the selection: two candidates of the first sequence taken as valid
    first = np.unique(at[:, 0] * n + at[:, 1], return_index=True)[1]
    v = want[first]
    seq2 = np.concatenate([[0, 0], seq[half:][first]]).astype(np.int32)
    pos2 = np.concatenate([[0, 2], pos[half:][first]]).astype(np.int32)
    tok2 = np.concatenate([[idx[between]] * 2, tok[half:][first]]).astype(np.int32)
    conf = rng.random(len(seq2), dtype=np.float32)
    want_s, _, st = oracle_lib.select(p, x, seq2[2:], pos2[2:], tok2[2:], conf[2:], v, NTH)
    sel, _ = g.select(x, seq2, pos2, tok2, conf, np.concatenate([[1, 1], v]).astype(np.uint8))
    assert st == 0 and g.errors() & ~(buffer | ENTRIES) == epic.DEV_CAPACITY
    assert not sel[:2].any() and np.array_equal(sel[2:], want_s)
