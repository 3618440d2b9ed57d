"""Tokens for a batch of host matchers that arrive while the fill before is still running: they are parsed beside it, and if it
turns out to have left pairs undecided the call fails and the matchers are where they were.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ALTS = " | ".join(f"r{i}" for i in range(20))
EBNF = ('root ::= "(" list ")"?\nlist ::= item ("," item)*\nitem ::= ' + ALTS + ' | "(" list ")"\n'
        + "".join(f'r{i} ::= "a"{{{i + 1}}} "b"*\n' for i in range(20)))
TOKS = [b"", b"(", b")", b",", b"a", b"b", b"ab,a", b"a,a", b"b,aa", b"b,a", b"ab", b"a,(", b"b),a", b"x"]


@pytest.fixture(scope="module")
def xg():
    import torch
    assert torch.cuda.is_available()
    import paper_2601_04426_amd as xg
    return xg


def _busy(torch):
    """A few milliseconds of work on the current stream, so that what is enqueued behind it has not begun when the host goes on."""
    a = torch.randn((4096, 4096), device="cuda:0")
    for _ in range(16):
        a = a @ a
        a /= a.abs().max()
    return a


# 3: one part, by the calling thread; 100: several parts, by the host threads
@pytest.mark.parametrize("B", [3, 100])
@pytest.mark.parametrize("undecided", [False, True])
def test_accept_beside_a_running_fill(xg, B, undecided):
    import torch
    vocab = xg.Vocab(TOKS, 0, [0])
    va = oracle.VocabArrays(TOKS, 0, [0])
    stream = torch.cuda.current_stream().cuda_stream
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=stream)
    orc = oracle.Oracle(EBNF, "root")
    ms = [xg.Matcher(cache) for _ in range(B)]
    batch = xg.MatcherBatch(ms)
    bm = torch.zeros((B, vocab.words), dtype=torch.int32, device="cuda:0")
    hist = []
    for b, m in enumerate(ms):
        for t in (b"(", b"a") if b % 3 != 2 else (b"(",):
            assert m.accept_token(TOKS.index(t))
        hist.append(b"(a" if b % 3 != 2 else b"(")
    # the end of the sequence, an accepted token, a rejected one, no token
    ids = np.array([[0, TOKS.index(b"b,a"), TOKS.index(b"x"), -1][b % 4] for b in range(B)], dtype=np.int32)
    ok = [np.unpackbits(oracle.pack_bitmask(orc.mask(h, va)).view(np.uint8), bitorder="little") for h in hist]
    want_status = np.array([0 if i < 0 or ok[b][i] else -3 for b, i in enumerate(ids)], dtype=np.int32)
    xg.fill_next_token_bitmask(batch, bm.data_ptr(), vocab.words, stream)       # what the library allocates for such a batch is there
    torch.cuda.synchronize()
    try:
        if undecided:
            xg.debug_set_large_capacity(8, 12)
        keep = _busy(torch)
        xg.fill_next_token_bitmask(batch, bm.data_ptr(), vocab.words, stream)
        filled = torch.cuda.Event()
        filled.record()
        assert not filled.query()               # the fill has not ended: the tokens below are parsed beside it
        if undecided:
            with pytest.raises(xg.Xg2Error) as err:
                batch.accept_tokens(ids)
            assert err.value.code == -4 and "undecided" in str(err.value)
            assert not any(m.is_terminated() for m in ms)
            # where they were: the pairs (if the list has room for all) are decided as for the state the fill saw, and so is another fill
            if B == 3:
                assert xg.fill_resolve_overflow(ms, bm.data_ptr(), vocab.words) > 0
            else:
                xg.debug_set_large_capacity(0, 0)
                xg.fill_next_token_bitmask(batch, bm.data_ptr(), vocab.words, stream)
            got = bm.cpu().numpy()
            for b in range(B):
                assert np.array_equal(got[b], oracle.pack_bitmask(orc.mask(hist[b], va))), b
        else:
            assert np.array_equal(batch.accept_tokens(ids), want_status)
        del keep
    finally:
        xg.debug_set_large_capacity(0, 0)
    if undecided:
        assert np.array_equal(batch.accept_tokens(ids), want_status)
    torch.cuda.synchronize()
    xg.fill_next_token_bitmask(batch, bm.data_ptr(), vocab.words, stream)
    got = bm.cpu().numpy()
    for b in range(B):
        if ids[b] == 0 and want_status[b] == 0:
            assert ms[b].is_terminated()
            continue
        h = hist[b] + (TOKS[ids[b]] if ids[b] > 0 and want_status[b] == 0 else b"")
        assert np.array_equal(got[b], oracle.pack_bitmask(orc.mask(h, va))), b
