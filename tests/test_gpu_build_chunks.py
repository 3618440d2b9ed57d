"""Chunks of a build: planes whose ranges of tokens end at, before and behind the edges of chunks and of what one thread cuts."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xg():
    import torch
    assert torch.cuda.is_available()
    import paper_2601_04426_amd as xg
    return xg


# (tokens that start with "a", rules): 64 ranks a chunk (a range at its edges; one thread's 32 chunks) and, beyond 8,192 full
# chunks in the launch, 128
@pytest.mark.parametrize("n,rules", [(1, 2), (63, 2), (64, 2), (65, 2), (127, 2), (128, 2), (129, 2), (2047, 2), (2048, 2), (2049, 2), (4161, 2), (4161, 320)])
def test_planes(xg, n, rules):
    letters = "abcdefg("
    toks, k = [b"<eos>", b"b", b")"], 0
    while len(toks) < n + 3:                                     # "a" and the digits of k to the base 8, as letters
        s, x = "", k
        while x:
            s, x = letters[x % 8] + s, x // 8
        toks.append(b"a" + s.encode())
        k += 1
    vocab, va = xg.Vocab(toks, 0, [0]), oracle.VocabArrays(toks, 0, [0])
    # a walk that defers to the recogniser, leaves rules early and nests; with many rules, planes of their own by what follows
    ebnf = "root ::= %s\n" % " | ".join("r%d" % r for r in range(rules))
    ebnf += "".join('r%d ::= [a-d]+ p%s "%s"\n' % (r, "?" if r % 2 else "", "".join(letters[(r >> s) & 7] for s in (0, 3, 6))) for r in range(rules))
    ebnf += 'p ::= "(" [a-g]* p? ")"\n'
    orc, cache = oracle.Oracle(ebnf, "root"), xg.compile_grammar(vocab, ebnf, "root")
    planes = cache.num_planes()
    assert rules == 2 or planes * (n // 128) > 8192, planes
    for k in range(0, planes, 1 if rules == 2 else 37):
        acc, unc = cache.get_planes(k)
        pos, parent = cache.plane_info(k)
        cls = orc.classes(pos, va, parent=parent, follow=True)
        assert np.array_equal(acc, oracle.pack_bitmask(cls == oracle.ACCEPTED)), ("accepted", k, pos, parent)
        assert np.array_equal(unc, oracle.pack_bitmask(cls == oracle.UNCERTAIN)), ("uncertain", k, pos, parent)
