"""Accepting tokens with planes under sites: several items of one rule instance (an entry that two items wait at), and contexts
and tokens around what lies across 64 lanes.  Statuses and masks against the oracle's plain definition; tolerance 0."""
import random

import numpy as np
import pytest

import oracle
from helpers import diff_words

pytestmark = pytest.mark.gpu

# after a letter an instance of `x` is both inside its own letters and behind a `y`: two items with one origin and one rule
EBNF = ('root ::= p\n'
        'p ::= "(" (p | x | q) ")"\n'
        'q ::= "[" (x | p) "]"\n'
        'x ::= [a-z]* | y "!" | y "?" y\n'
        'y ::= [a-z]+ | "{" x "}"\n')


@pytest.mark.parametrize("depths", [(1, 2, 3, 5), (14, 15, 16, 20), (29, 30, 31, 32), (45, 46, 47, 48), (58, 59, 60, 61, 62, 63, 64, 65, 70)])
def test_several_items_and_deep_contexts(depths):
    import torch
    import paper_2601_04426_amd as xg
    stream = torch.cuda.current_stream().cuda_stream
    toks = [b""] + [bytes([c]) for c in b"()[]{}!?abz"] + [b"((", b"ab", b"b!", b"z)", b"}!)", b"abz?ab", b"(([", b"{ab", b"{a}!)", b"))", b")))", b"abzabzabzabzabzz", b"abzabzabzabzabzab"]
    vocab, va = xg.Vocab(toks, 0, [0]), oracle.VocabArrays(toks, 0, [0])
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=stream)
    orc = oracle.Oracle(EBNF, "root")
    starts = [b"(" * d + tail for d in depths for tail in (b"a", b"[ab", b"{z", b"{a}?b")]
    B, W = len(starts), vocab.words
    db = xg.DeviceBatch(vocab, B)
    db.assign(cache, stream=stream)
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    bitmask = torch.full((B, W), -1, dtype=torch.int32, device="cuda")
    hist, rng = [b""] * B, random.Random(depths[0])

    def accept(nxt):
        ids = torch.tensor(nxt, dtype=torch.int32, device="cuda")
        db.accept_tokens(ids.data_ptr(), status.data_ptr(), stream)
        assert not status.cpu().numpy().any(), (hist, nxt)
        for b, t in enumerate(nxt):
            if t > 0:
                hist[b] += toks[t]

    for k in range(max(len(s) for s in starts)):
        accept([toks.index(s[k:k + 1]) if k < len(s) else -1 for s in starts])
    for step in range(6):
        db.fill_next_token_bitmask(bitmask.data_ptr(), W, stream)
        got = bitmask.cpu().numpy()
        nxt = []
        for b in range(B):
            allowed = orc.mask(hist[b], va)
            want = oracle.pack_bitmask(allowed)
            assert np.array_equal(got[b], want), (step, b, hist[b], diff_words(got[b], want, toks))
            can = [int(t) for t in np.nonzero(allowed)[0] if t != 0]
            nxt.append(max(rng.sample(can, min(3, len(can))), key=lambda t: len(toks[t])) if can else -1)
        refused = [next((int(t) for t in range(1, len(toks)) if not orc.mask(hist[b], va)[t]), -1) for b in range(B)]
        ids = torch.tensor(refused, dtype=torch.int32, device="cuda")
        db.accept_tokens(ids.data_ptr(), status.data_ptr(), stream)
        assert (status.cpu().numpy() == np.where(np.array(refused) < 0, 0, -3)).all()
        accept(nxt)
