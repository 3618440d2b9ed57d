"""The ways a row's uncertain tokens can take through a fill (a wavefront each, a lane each, word by word) where the tokens or
their item sets do not fit a lane's lists: same masks, same counts, and no way that costs many times another."""
import random

import numpy as np
import pytest

import oracle
from helpers import diff_words

pytestmark = pytest.mark.gpu

# the token of an `x` ends it and closes parentheses: which closers fit depends on the context, so with planes of single
# positions and no follow filter every token of letters and closers is uncertain
EBNF = ('root ::= p | b\n'
        'p ::= "(" (p | b | x) ")"\n'
        'b ::= "[" (p | b | x) "]"\n'
        'x ::= [a-z]+\n')


def _stream():
    import torch
    return torch.cuda.current_stream().cuda_stream


@pytest.fixture(scope="module")
def xg():
    import torch
    assert torch.cuda.is_available()
    import paper_2601_04426_amd as xg
    return xg


def _tokens(n_uncertain, shortest, longest):
    toks = [b""] + [bytes([c]) for c in b"()[]abz"]
    rng, have = random.Random(n_uncertain), set(toks)
    while len(toks) < 8 + n_uncertain:
        n = rng.randint(shortest, longest)
        k = rng.randint(1, min(n - 1, 12))
        t = bytes(rng.choice(b"abz") for _ in range(n - k)) + bytes(rng.choice(b"))])") for _ in range(k))
        if t not in have:
            have.add(t)
            toks.append(t)
    return toks


def _batch(xg, toks, starts, ebnf=EBNF):
    """Slots that have seen `starts`, on the device."""
    import torch
    vocab = xg.Vocab(toks, 0, [0])
    cache = xg.compile_grammar(vocab, ebnf, "root", stream=_stream(), context_depth=1, follow_filter=False)
    B = len(starts)
    db = xg.DeviceBatch(vocab, B)
    db.assign(cache, stream=_stream())
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    for k in range(max(len(s) for s in starts)):
        ids = torch.tensor([toks.index(s[k:k + 1]) if k < len(s) else -1 for s in starts], dtype=torch.int32, device="cuda")
        db.accept_tokens(ids.data_ptr(), status.data_ptr(), _stream())
        assert not status.cpu().numpy().any()
    return vocab, cache, db


@pytest.mark.parametrize("n", [6, 24, 25, 63, 64, 100])
def test_count_of_large_tokens_does_not_depend_on_the_way(xg, n):
    """Every uncertain token is longer than a lane takes: all are counted, rejected ones too."""
    import torch
    starts = [b"(" * 8 + b"z"] * 5
    vocab, cache, db = _batch(xg, _tokens(n, 17, 40), starts)
    bm = torch.zeros((len(starts), vocab.words), dtype=torch.int32, device="cuda")
    db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream())
    assert xg.fill_last_recheck_tokens(len(starts)).tolist() == [n] * len(starts)
    assert xg.fill_last_status() == (len(starts) * n, False)


# a rule that one of twelve rules or another instance of itself can stand in: entering it brings more than a lane's list holds
WIDE = ('root ::= p\np ::= "(" (p | ' + " | ".join("r%d" % k for k in range(12)) + ') ")"\n'
        + "".join('r%d ::= "%s" [a-z]*\n' % (k, "abz"[k % 3] * (1 + k // 3)) for k in range(12)))


@pytest.mark.parametrize("rows", [1, 20, 65])                         # times eight or three; the last beyond kFillSpreadRows
@pytest.mark.parametrize("ebnf,n,shortest,longest", [
    (EBNF, 18, 9, 40), (EBNF, 19, 17, 40), (EBNF, 24, 9, 40), (EBNF, 48, 9, 40), (EBNF, 49, 17, 64),
    (EBNF, 6, 65, 80), (EBNF, 7, 65, 80), (EBNF, 18, 60, 80), (EBNF, 19, 60, 80), (EBNF, 25, 9, 80),         # beyond what a wavefront takes
    (EBNF, 63, 17, 40), (EBNF, 64, 17, 40), (EBNF, 600, 9, 80),       # a plane's list, and more
    (WIDE, 24, 4, 16), (WIDE, 40, 4, 16), (WIDE, 100, 4, 24),         # item sets that outgrow a lane
], ids=lambda v: "wide" if v is WIDE else "nest" if v is EBNF else str(v))
def test_masks_with_large_tokens(xg, ebnf, n, shortest, longest, rows):
    import torch
    toks = _tokens(n, shortest, longest)
    # contexts around 64 sets and 128 wait entries, and (on the host) beyond the 512 entries and 240 sets of a matcher slot
    depths = [1, 8, 42, 43, 63, 64, 65, 118] if ebnf is EBNF else [1, 5, 12]
    starts = [b"(" * d + b"z" for d in depths]
    deep = [b"(" * d + b"z" for d in (175, 245)]
    orc, va = oracle.Oracle(ebnf, "root"), oracle.VocabArrays(toks, 0, [0])
    want = {s: oracle.pack_bitmask(orc.mask(s, va)) for s in starts + deep}
    vocab, cache, db = _batch(xg, toks, starts * rows, ebnf)
    W = vocab.words

    def check(fill, hist):
        bm = torch.full((len(hist), W), -1, dtype=torch.int32, device="cuda")
        fill(bm)
        assert not xg.fill_last_status()[1]
        torch.cuda.synchronize()
        got = bm.cpu().numpy()
        for b, s in enumerate(hist):
            assert np.array_equal(got[b], want[s]), (b, s, diff_words(got[b], want[s], toks))

    for _ in range(2):
        check(lambda bm: db.fill_next_token_bitmask(bm.data_ptr(), W, _stream()), starts * rows)
    at = {t: k for k, t in enumerate(toks)}
    for hist in (starts * rows, deep * rows + starts):
        matchers = [xg.Matcher(cache) for _ in hist]
        for m, s in zip(matchers, hist):
            for c in s:
                assert m.accept_token(at[bytes([c])])
        check(lambda bm: xg.fill_next_token_bitmask(matchers, bm.data_ptr(), W, _stream()), hist)
        if rows > 20:                                                 # (a deep context for each would not fit its staging area)
            continue
        few = matchers[:128]                                          # the most rows that its fixed scratch has lanes of their own for;
        #                                                               with 600 tokens a row they fill its overflow list
        check(lambda bm: xg.fill_next_token_bitmask_noalloc(few, bm.data_ptr(), W, _stream()), hist[:128])


def _apart(toks, n):
    """Tokens that are nowhere allowed (no rule reads a "#") behind every token of more than a byte: ids n apart."""
    out = []
    for t in toks:
        out.append(t)
        if len(t) > 1:
            out += [b"#%d" % (len(out) + k) for k in range(n - 1)]
    return out


def _matchers(xg, cache, toks, hist):
    at = {t: k for k, t in enumerate(toks)}
    matchers = [xg.Matcher(cache) for _ in hist]
    for m, s in zip(matchers, hist):
        for c in s:
            assert m.accept_token(at[bytes([c])])
    return matchers


# rows, uncertain tokens: with two, four and six lanes of the large-capacity scratch for each row, fewer than the row has
# wavefronts that take candidate words (here more of them than 16 for each wavefront)
@pytest.mark.parametrize("rows,n,apart", [(128, 600, 16), (64, 1100, 8), (42, 1700, 8)])
def test_full_list_and_candidates_far_apart(xg, rows, n, apart):
    """More large tokens than the overflow list of the call that allocates nothing holds, from words that all wavefronts have a share of."""
    import torch
    toks = _apart(_tokens(n, 17, 40), apart)
    kinds = [b"(" * d + b"z" for d in (1, 8, 42, 43, 63, 64, 65, 118)]
    starts = [kinds[k % len(kinds)] for k in range(rows)]
    orc, va = oracle.Oracle(EBNF, "root"), oracle.VocabArrays(toks, 0, [0])
    want = {s: oracle.pack_bitmask(orc.mask(s, va)) for s in kinds}
    vocab = xg.Vocab(toks, 0, [0])
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=_stream(), context_depth=1, follow_filter=False)
    matchers, W = _matchers(xg, cache, toks, starts), vocab.words
    for _ in range(2):
        bm = torch.full((rows, W), -1, dtype=torch.int32, device="cuda")
        xg.fill_next_token_bitmask_noalloc(matchers, bm.data_ptr(), W, _stream())
        assert xg.fill_last_status() == (rows * n, False) and rows * n > 1 << 16
        got = bm.cpu().numpy()
        for b, s in enumerate(starts):
            assert np.array_equal(got[b], want[s]), (b, s, diff_words(got[b], want[s], toks))


@pytest.mark.parametrize("rows", [1, 24, 300])
def test_large_tokens_of_a_plane_built_by_the_fill(xg, rows):
    """Nobody has counted the plane's uncertain tokens when the fill is launched: it has more than its list holds, and no launch behind."""
    import torch
    toks = _apart(_tokens(3000, 17, 40), 4)
    kinds = [b"(" * d + b"z" for d in (2, 9, 30, 61)]
    starts = [kinds[k % len(kinds)] for k in range(rows)]
    orc, va = oracle.Oracle(EBNF, "root"), oracle.VocabArrays(toks, 0, [0])
    want = {s: oracle.pack_bitmask(orc.mask(s, va)) for s in kinds}
    vocab = xg.Vocab(toks, 0, [0])
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=_stream(), jit=True, jit_prebuild=0)
    matchers, W = _matchers(xg, cache, toks, starts), vocab.words
    for _ in range(2):                                               # while the plane is built, and when it is counted
        bm = torch.full((rows, W), -1, dtype=torch.int32, device="cuda")
        xg.fill_next_token_bitmask(matchers, bm.data_ptr(), W, _stream())
        assert min(xg.fill_last_recheck_tokens(rows)) > 12 * 16 * 2 and not xg.fill_last_status()[1]
        got = bm.cpu().numpy()
        for b, s in enumerate(starts):
            assert np.array_equal(got[b], want[s]), (b, s, diff_words(got[b], want[s], toks))


# two rules for the same text: every uncertain token is a candidate twice
TWICE = ('root ::= p | b\n'
         'p ::= "(" (p | b | x | y) ")"\n'
         'b ::= "[" (p | b | x) "]"\n'
         'x ::= [a-z]+\n'
         'y ::= [a-z]+ "."?\n')


@pytest.mark.parametrize("rows", [1, 256, 257, 512, 513, 600, 1024, 1025])  # a workgroup of 16 wavefronts, or of 12 or 6
@pytest.mark.parametrize("ebnf,n", [(EBNF, 2), (EBNF, 3), (EBNF, 24), (EBNF, 25), (EBNF, 32), (EBNF, 33), (EBNF, 42), (EBNF, 43), (EBNF, 48), (EBNF, 49),
                                    (EBNF, 63), (TWICE, 12), (TWICE, 13), (TWICE, 24), (TWICE, 25), (TWICE, 32), (TWICE, 33), (TWICE, 43), (TWICE, 60)],
                         ids=lambda v: "twice" if v is TWICE else "nest" if v is EBNF else str(v))
def test_masks_by_size_of_the_workgroup(xg, ebnf, n, rows):
    """Up to four candidates for each wavefront of a row, and more: 24, 48, 64 and the next of each, in a row's one plane or in two;
    planes on both sides of the lines that decide on the number of wavefronts (2, 24, 32 and 42 tokens)."""
    import torch
    toks = _tokens(n, 3, 14)
    kinds = [b"(", b"(z", b"([z", b"((((b", b"(" * 12 + b"a"]
    starts = [kinds[(k * 7) % len(kinds)] for k in range(rows)]
    vocab, cache, db = _batch(xg, toks, starts, ebnf)
    orc, va = oracle.Oracle(ebnf, "root"), oracle.VocabArrays(toks, 0, [0])
    want = {s: oracle.pack_bitmask(orc.mask(s, va)) for s in set(starts)}
    bm = torch.full((rows, vocab.words), -1, dtype=torch.int32, device="cuda")
    for _ in range(2):
        db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream())
        assert not xg.fill_last_status()[1]
        assert np.array_equal(bm.cpu().numpy(), np.stack([want[s] for s in starts]))


@pytest.mark.parametrize("rows", [2, 300])
@pytest.mark.parametrize("V", [131071, 131072 + 33, 163840, 163840 + 1])
def test_masks_of_rows_beyond_one_block(xg, V, rows):
    """The union asks for 4,096 or 5,120 words of a row at a time: rows of that many and a few more."""
    import itertools
    import torch
    toks = [b""] + [bytes([c]) for c in b"()[]"]
    for n in (1, 2, 3, 4):
        toks += [bytes(t) for t in itertools.islice(itertools.product(b"abcdefghijklmnopqrstuvwxyz", repeat=n), V - len(toks) - 2)]
    toks += [b"zz)", b"a]"]
    assert len(toks) == V and len(set(toks)) == V
    starts = [[b"(z", b"[", b"([", b""][k % 4] for k in range(rows)]
    vocab, cache, db = _batch(xg, toks, starts)
    orc, va = oracle.Oracle(EBNF, "root"), oracle.VocabArrays(toks, 0, [0])
    want = {s: oracle.pack_bitmask(orc.mask(s, va)) for s in set(starts)}
    bm = torch.full((rows, vocab.words), -1, dtype=torch.int32, device="cuda")
    db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream())
    assert np.array_equal(bm.cpu().numpy(), np.stack([want[s] for s in starts]))


def _us(f):
    import torch
    f()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 5)
    return best


def test_large_tokens_are_not_parsed_one_after_another(xg):
    """A row's tokens beyond a lane's lists, on either side of what a plane's list holds (63): within small factors of tokens that
    fit, measured 2.4 and 3; one after another they took 8 and 130 times as long."""
    import torch

    def us(n, shortest, longest):
        vocab, _, db = _batch(xg, _tokens(n, shortest, longest), [b"(" * 8 + b"z"])
        bm = torch.zeros((1, vocab.words), dtype=torch.int32, device="cuda")
        return _us(lambda: db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream()))

    fit = us(63, 9, 14)
    assert us(63, 20, 40) < 5 * fit
    assert us(100, 20, 40) < 10 * fit


def test_neighbouring_candidates_are_spread_over_the_row(xg):
    """300 tokens in ten mask words, one row: measured 2.7 times as long as the 63 that a plane's list holds; 16 times where
    one wavefront took all ten words."""
    import torch

    def us(n):
        vocab, _, db = _batch(xg, _tokens(n, 3, 14), [b"(" * 8 + b"z"])
        bm = torch.zeros((1, vocab.words), dtype=torch.int32, device="cuda")
        return _us(lambda: db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream()))

    few, many = us(63), us(300)
    print("us: %.1f, %.1f" % (few, many))
    assert many < 5 * few


def test_captured_fill(xg):
    """Replays of one captured fill whose rows leave tokens to the launch behind it: each as if it were the first."""
    import torch
    toks, starts = _tokens(100, 17, 40), [b"(" * 8 + b"z", b"(" * 3 + b"a", b"[([(" + b"b"]
    vocab, cache, db = _batch(xg, toks, starts)
    orc, va = oracle.Oracle(EBNF, "root"), oracle.VocabArrays(toks, 0, [0])
    want = np.stack([oracle.pack_bitmask(orc.mask(s, va)) for s in starts])
    bm = torch.zeros((len(starts), vocab.words), dtype=torch.int32, device="cuda")
    db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream())
    torch.cuda.synchronize()
    once = xg.fill_last_status()
    assert once == (3 * 100, False)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        db.fill_next_token_bitmask(bm.data_ptr(), vocab.words, _stream())
    for _ in range(4):
        bm.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bm.cpu().numpy(), want)
        assert xg.fill_last_status() == once
