"""A batch whose slots' wait entries take more than 4 GiB: every slot's states and masks are its own.  Tolerance 0."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

EBNF = ('root ::= p | b\n'
        'p ::= "(" (p | b | x) ")"\n'
        'b ::= "[" (p | b | x) "]"\n'
        'x ::= [a-z]+\n')
SLOT_WAITS, MOST = 512 * 8, 1 << 20                                   # bytes of a slot's wait entries in one of its two buffers; slots accepted


def test_states_beyond_4_gib():
    import torch
    import paper_2601_04426_amd as xg
    stream = torch.cuda.current_stream().cuda_stream
    toks = [b""] + [bytes([c]) for c in b"()[]abz"] + [b"))", b")]", b"])", b"]]", b"z))", b"z)]", b"z])", b"z]]", b"a)))", b"((", b"[(a", b"ab"]
    at = {t: k for k, t in enumerate(toks)}
    B = MOST // 2 + 300                                               # the last 300 slots' second buffers lie behind 4 GiB,
    first = MOST - B                                                  #   from this slot on: with 32 bits the same entries as slots 0 .. 599
    assert (B + first) * SLOT_WAITS == 1 << 32
    kinds = [b"(z", b"([z", b"[((a", b"[[[[b", b"((((([z"]
    kind = np.arange(B) * 7 % len(kinds)
    assert (kind[first:] != kind[:B - first]).all()
    vocab, va = xg.Vocab(toks, 0, [0]), oracle.VocabArrays(toks, 0, [0])
    orc, cache = oracle.Oracle(EBNF, "root"), xg.compile_grammar(vocab, EBNF, "root", stream=stream)
    W = vocab.words
    db = xg.DeviceBatch(vocab, B)
    db.assign(cache, stream=stream)
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    bitmask = torch.full((B, W), -1, dtype=torch.int32, device="cuda")
    hist = [b""] * len(kinds)

    def accept(ids, want):
        db.accept_tokens(torch.from_numpy(np.array(ids, dtype=np.int32)[kind]).cuda().data_ptr(), status.data_ptr(), stream)
        got = status.cpu().numpy()
        assert (got == want).all(), (ids, np.nonzero(got != want)[0][:8])

    def masks():
        bitmask.fill_(-1)
        db.fill_next_token_bitmask(bitmask.data_ptr(), W, stream)
        got, allowed = bitmask.cpu().numpy(), [orc.mask(h, va) for h in hist]
        want = np.stack([oracle.pack_bitmask(a) for a in allowed])[kind]
        assert np.array_equal(got, want), (hist, np.nonzero((got != want).any(axis=1))[0][:8])
        return allowed

    for k in range(max(len(s) for s in kinds)):                       # (slots change buffers with every token)
        accept([at[s[k:k + 1]] if k < len(s) else -1 for s in kinds], 0)
        hist = [s[:k + 1] for s in kinds]
    for _ in range(4):
        allowed = masks()
        accept([next(t for t in range(1, len(toks)) if not a[t]) for a in allowed], -3)
        ids = [max((t for t in range(1, len(toks)) if a[t]), key=lambda t: (toks[t].count(b")") + toks[t].count(b"]"), t), default=-1) for a in allowed]
        accept(ids, 0)
        hist = [h + (toks[t] if t > 0 else b"") for h, t in zip(hist, ids)]
    masks()
