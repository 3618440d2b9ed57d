"""Fill and accept where the wavefront-wide parse changes its way: numbers of candidates around what a wavefront each, a
lane each and the planes' lists take; contexts and tokens around what fits across 64 lanes.  Masks against the oracle's
plain definition, for matchers on the host and on the device; tolerance 0.
"""
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


def _tokens(n_uncertain, lengths):
    toks = [b""] + [bytes([c]) for c in b"()[]abz"] + [b"((", b"[(", b"((((((((", b"zz"]
    rng = random.Random(n_uncertain)
    want = len(toks) + n_uncertain
    while len(toks) < want:
        n = rng.choice(lengths)
        k = rng.randint(1, min(n - 1, 12))
        t = bytes(rng.choice(b"abz") for _ in range(n - k)) + bytes(rng.choice(b"))])") for _ in range(k))
        if t not in toks:
            toks.append(t)
    return toks


@pytest.mark.parametrize("n_uncertain,lengths", [
    (1, (4,)), (24, (8, 16)), (25, (8, 16)),              # a wavefront each, up to four in turn
    (24, (15, 16, 17, 48, 63, 64, 65, 70)),               # token lengths: a vector load, a wavefront's bytes, beyond
    (25, (15, 16, 17, 48, 63, 64, 65, 70)), (48, (15, 16, 17, 48, 63, 64, 65, 70)), (49, (15, 16, 17, 48, 63, 64, 65, 70)),
    (63, (12,)), (64, (12, 20)),                          # the length of a plane's list, and one more
    (600, (9, 12)),                                       # more than the row's list
])
def test_masks_at_the_edges_of_the_parse(xg, n_uncertain, lengths):
    import torch
    dev = torch.device("cuda:0")
    toks = _tokens(n_uncertain, lengths)
    vocab, va = xg.Vocab(toks, 0, [0]), oracle.VocabArrays(toks, 0, [0])
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=_stream(), context_depth=1, follow_filter=False)
    orc = oracle.Oracle(EBNF, "root")
    rng = random.Random(7)
    # nesting depths around 64 item sets, and 64 and 128 wait entries, of a row's context
    starts = ([b""] + [b"(" * d + b"z" for d in (1, 2, 8, 14, 15, 16, 20, 21, 22, 30, 31, 32, 40, 46, 47, 48, 60, 61, 62, 63, 64, 65, 70)]
              + [b"[(" * d + b"ab" for d in (1, 10, 31, 32, 40)])
    B, W = len(starts), vocab.words
    single = {t[0]: i for i, t in enumerate(toks) if len(t) == 1}
    hist = [b""] * B
    matchers = [xg.Matcher(cache) for _ in range(B)]
    db = xg.DeviceBatch(vocab, B)
    db.assign(cache, stream=_stream())
    ids, status = torch.zeros(B, dtype=torch.int32, device=dev), torch.zeros(B, dtype=torch.int32, device=dev)
    bm_host, bm_dev = (torch.full((B, W), -1, dtype=torch.int32, device=dev) for _ in range(2))

    def accept(nxt):
        ids.copy_(torch.tensor(nxt, dtype=torch.int32))
        db.accept_tokens(ids.data_ptr(), status.data_ptr(), _stream())
        assert not status.cpu().numpy().any(), (hist, nxt)
        for b, t in enumerate(nxt):
            if t > 0:
                assert matchers[b].accept_token(t)
                hist[b] += toks[t]

    for k in range(max(len(s) for s in starts)):
        accept([single[s[k]] if k < len(s) else -1 for s in starts])
    most = 0
    for step in range(5):
        xg.fill_next_token_bitmask(matchers, bm_host.data_ptr(), W, _stream())
        most = max(most, int(xg.fill_last_recheck_tokens(B).max()))
        assert not xg.fill_last_status()[1]
        db.fill_next_token_bitmask(bm_dev.data_ptr(), W, _stream())
        assert not xg.fill_last_status()[1]
        torch.cuda.synchronize()
        got_host, got_dev = bm_host.cpu().numpy(), bm_dev.cpu().numpy()
        nxt = []
        for b in range(B):
            allowed = orc.mask(hist[b], va)
            want = oracle.pack_bitmask(allowed)
            assert np.array_equal(got_host[b], want), ("host", step, b, hist[b], diff_words(got_host[b], want, toks))
            assert np.array_equal(got_dev[b], want), ("device", step, b, hist[b], diff_words(got_dev[b], want, toks))
            can = [int(t) for t in np.nonzero(allowed)[0] if t != 0]
            nxt.append(max(rng.sample(can, min(3, len(can))), key=lambda t: len(toks[t])) if can else -1)
        accept(nxt)
    assert most >= n_uncertain                                        # every one of them went through the re-check somewhere
