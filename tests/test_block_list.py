"""Device blocks kept between requests (`csrc/block_list.hpp`) on the host, under AddressSanitizer and UndefinedBehaviorSanitizer:
which blocks are handed out again and when, with memory that counts what is taken and can refuse to wait."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "hostcheck", "block_list_main.cpp")


def test_blocks_kept_between_requests(tmp_path):
    exe = str(tmp_path / "block_list_main")
    cmd = ["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-o", exe, SRC]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    env.pop("LD_PRELOAD", None)
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=60)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout[-3000:]


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["relaxed", "thread_local"])
def test_destroying_beside_a_capture(mode):
    """A cache and its pool destroyed while a stream is captured (by the same thread in relaxed mode, by another in
    thread-local mode) leave the capture whole, and what is compiled into their memory afterwards is right."""
    import threading

    import numpy as np
    import torch

    import gen
    import paper_2601_04426_amd as xg

    v = gen.make_vocab(2048, 11, "tiny")
    vocab = xg.Vocab(v.tokens, v.eos_id, v.special_ids)
    ebnf = 'root ::= "[" ws item (ws "," ws item){0,20} ws "]"\nitem ::= "\\"" [a-z]{0,30} "\\"" | "-"? [0-9]{1,9}\nws ::= [ \\n]*\n'

    def planes(cache):
        return [cache.get_planes(k) for k in range(cache.num_planes())]

    stream = torch.cuda.Stream()
    caches = [xg.compile_grammar(vocab, ebnf, stream=stream.cuda_stream)]
    want = planes(caches[0])
    x = torch.zeros(1024, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode=mode):
        x += 1
        if mode == "relaxed":
            caches.clear()
        else:
            t = threading.Thread(target=caches.clear)
            t.start()
            t.join()
        x += 1
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert x.eq(2.0 * (k + 1)).all()
    again = xg.compile_grammar(vocab, ebnf)
    for (a, u), (a2, u2) in zip(want, planes(again)):
        assert np.array_equal(a, a2) and np.array_equal(u, u2)
