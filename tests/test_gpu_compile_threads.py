"""Rules analysed on host threads: planes of grammars on both sides of the line, also while other threads compile and accept."""
import random
import threading

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xg():
    import torch
    assert torch.cuda.is_available()
    import paper_2601_04426_amd as xg
    return xg


def _calls(n_rules: int, length: int, seed: int) -> str:
    """One rule a call: a literal, a choice, an optional part and a reference, about `length` + 12 states."""
    rng = random.Random(seed)
    word = lambda n: "".join(rng.choice("abcde") for _ in range(n))  # noqa: E731
    lines = ["root ::= " + " | ".join("r%d" % k for k in range(n_rules)), "opt ::= \"\" | \" \" opt"]
    for k in range(n_rules):
        lines.append('r%d ::= "%s" opt ("%s" | "%s")? "%s%d"' % (k, word(length), word(3), word(5), word(4), k))
    return "\n".join(lines) + "\n"


def _planes(cache):
    return [(cache.plane_info(k), [p.tobytes() for p in cache.get_planes(k)]) for k in range(cache.num_planes())]


@pytest.mark.parametrize("n_rules,length", [(3, 20), (30, 12), (34, 40), (80, 4)])    # 73 and 763 states besides the largest rule, 1,794 and 1,477
def test_planes(xg, n_rules, length):
    tok = gen.make_vocab(1500, 5, "bpe")
    vocab = xg.Vocab(tok.tokens, tok.eos_id, tok.special_ids)
    va = oracle.VocabArrays(tok.tokens, tok.eos_id, tok.special_ids)
    ebnf = _calls(n_rules, length, 7 * n_rules + length)
    orc = oracle.Oracle(ebnf, "root")
    cache = xg.compile_grammar(vocab, ebnf, "root")
    for k in range(0, cache.num_planes(), 3):
        acc, unc = cache.get_planes(k)
        pos, parent = cache.plane_info(k)
        cls = orc.classes(pos, va, parent=parent, follow=True)
        assert np.array_equal(acc, oracle.pack_bitmask(cls == oracle.ACCEPTED)), ("accepted", k)
        assert np.array_equal(unc, oracle.pack_bitmask(cls == oracle.UNCERTAIN)), ("uncertain", k)


def test_beside_other_threads(xg):
    """Two threads compile and one advances matchers in batches: every cache and every status is what one thread alone gets."""
    tok = gen.make_vocab(1500, 5, "bpe")
    vocab = xg.Vocab(tok.tokens, tok.eos_id, tok.special_ids)
    texts = [_calls(34, 40, 1), _calls(40, 30, 2)]
    want = [_planes(xg.compile_grammar(vocab, t, "root")) for t in texts]
    cfg = gen.build_config(1)
    ebnf, root = cfg.grammars[0]
    g, v = xg.Grammar(ebnf, root), xg.Vocab(cfg.vocab.tokens, 0, [0])
    seg, rng, B = gen.Segmenter(cfg.vocab), random.Random(3), 160
    traces = [seg.segment(cfg.sample_text(rng, 0), rng) for _ in range(B)]
    errors = []

    def compiles(k):
        try:
            for _ in range(3):
                assert _planes(xg.compile_grammar(vocab, texts[k], "root")) == want[k], k
        except Exception as e:                                   # reported by the main thread
            errors.append(repr(e)[:500])

    def accepts():
        try:
            for _ in range(4):
                batch = xg.MatcherBatch([xg.Matcher(grammar=g, vocab=v) for _ in range(B)])
                for step in range(8):
                    status = batch.accept_tokens([t[step] if step < len(t) else -1 for t in traces])
                    assert not np.asarray(status).any(), step
        except Exception as e:
            errors.append(repr(e)[:500])

    threads = [threading.Thread(target=compiles, args=(0,)), threading.Thread(target=compiles, args=(1,)), threading.Thread(target=accepts)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads), "a caller is stuck"
    assert not errors, errors
