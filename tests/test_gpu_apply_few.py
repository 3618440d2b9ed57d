"""Pieces of a row with few masked, or few allowed, tokens: their masked tokens are stored one by one where that is less than
reading, merging and writing vectors.  Around the numbers that decide on it, with rows at any place; bit for bit.
"""
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


def _masks(rng, W, kind, k):
    """[W] words: `few`: k masked tokens in some words; `most`: k allowed tokens in some; `whole`: masked halves of words, k masked besides."""
    out = np.full(W, 0xFFFFFFFF if kind != "most" else 0, dtype=np.uint32)
    for w in rng.choice(W, size=max(1, W // 3), replace=False):
        bits = rng.choice(16 if kind == "whole" else 32, size=min(k, 16), replace=False)
        m = np.uint32(sum(1 << int(b) for b in bits))
        out[w] = m if kind == "most" else ~m & np.uint32(0xFFFFFFFF)
        if kind == "whole":
            out[w] &= np.uint32(0x0000FFFF)
    return out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["few", "most", "whole"])
@pytest.mark.parametrize("V", [33, 2048, 2085, 6150])
def test_few_masked_or_allowed(xg, dtype, kind, V):
    import torch
    dev = torch.device("cuda:0")
    u, code = (np.uint32, xg.XG2_F32) if dtype == "f32" else (np.uint16, xg.XG2_BF16)
    size, W = np.dtype(u).itemsize, (V + 31) // 32
    rng = np.random.default_rng(V)
    counts = [1, 2, 3, 4, 5, 7, 8, 9, 12]
    bm = np.stack([_masks(rng, W, kind, k) for k in counts]).view(np.int32)
    bm_t = torch.from_numpy(bm).to(dev)
    B, stride = len(counts), V + 3
    for off in (0, size, 16, 128 - size):
        raw = rng.integers(0, 256, size=256 + B * stride * size + 256, dtype=np.uint8)
        t = torch.from_numpy(raw).to(dev)
        xg.apply_token_bitmask(t.data_ptr() + 128 + off, code, B, V, stride, bm_t.data_ptr(), W, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        want = raw.copy()
        rows = np.frombuffer(want[128 + off:128 + off + B * stride * size].tobytes(), dtype=u).reshape(B, stride).copy()
        part = np.ascontiguousarray(rows[:, :V])
        (oracle.apply_f32 if dtype == "f32" else oracle.apply_bf16)(part, bm)
        rows[:, :V] = part
        want[128 + off:128 + off + B * stride * size] = np.frombuffer(rows.tobytes(), dtype=np.uint8)
        assert np.array_equal(t.cpu().numpy(), want), off


# 64 and 256 MB: what counts as few changes there
@pytest.mark.parametrize("dtype,B,V", [("bf16", 220, 152001), ("bf16", 221, 152001), ("f32", 111, 150001), ("f32", 112, 150001), ("f32", 448, 150001)])
def test_few_in_large_logits(xg, dtype, B, V):
    import torch
    dev = torch.device("cuda:0")
    W = (V + 31) // 32
    tt, ninf = (torch.int16, -128) if dtype == "bf16" else (torch.int32, -8388608)     # 0xFF80, 0xFF800000
    g = torch.Generator(device=dev).manual_seed(B)
    logits = torch.randint(-2 ** 15, 2 ** 15, (B, V), generator=g, device=dev, dtype=tt)
    p = torch.tensor([0.0, 0.001, 0.02, 0.1, 0.9, 0.99, 0.999, 1.0], device=dev)[torch.arange(B, device=dev) % 8]
    masked = torch.rand((B, W * 32), generator=g, device=dev) < p[:, None]
    words = ((~masked).view(B, W, 32).long() << torch.arange(32, device=dev)).sum(-1)
    bm = torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32)
    want = logits.clone()
    want[masked[:, :V]] = ninf
    xg.apply_token_bitmask(logits.data_ptr(), xg.XG2_BF16 if dtype == "bf16" else xg.XG2_F32, B, V, V, bm.data_ptr(), W,
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(logits, want)
