"""The ways a row's uncertain tokens can take through a fill (a wavefront each, a lane each, word by word) where the tokens or
their item sets do not fit a lane's lists: same masks, same counts, and no way that costs many times another."""
import random

import pytest


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


def _batch(xg, toks, starts, **options):
    """Slots that have seen `starts`, on the device."""
    import torch
    vocab = xg.Vocab(toks, 0, [0])
    cache = xg.compile_grammar(vocab, EBNF, "root", stream=_stream(), context_depth=1, follow_filter=False, **options)
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
