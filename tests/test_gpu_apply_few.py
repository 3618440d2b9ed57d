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
@pytest.mark.parametrize("dtype,B,V", [("bf16", 220, 152001), ("bf16", 221, 152001), ("bf16", 884, 152001), ("f32", 111, 150001), ("f32", 112, 150001), ("f32", 448, 150001)])
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


def _pieces(rng):
    """[n, 64] words: pieces of 2,048 tokens around the numbers that decide how one is written, each three times with its words at other places:
    (words with single masked tokens, how many such tokens in all, what the other words hold) and (half masked words, words allowed as a
    whole, the others masked)."""
    few = [(w, t, rest) for w, t in [(1, 8), (1, 9), (8, 48), (8, 49), (14, 110), (14, 111), (16, 64), (16, 65), (16, 88), (16, 89), (16, 128), (20, 100), (20, 101),
                                     (20, 140), (20, 141), (32, 96), (32, 97), (39, 49), (39, 96), (39, 110), (39, 111), (40, 48), (40, 49), (48, 48), (49, 49),
                                     (64, 64), (64, 96), (64, 97), (64, 160), (64, 161), (64, 232), (64, 233), (64, 272), (64, 273), (60, 480)] for rest in (0xFFFFFFFF, 0)]
    half = [(n, o) for n in (38, 39, 40, 41, 56) for o in (0, 8, 9, 16, 17, 24, 25) if n + o <= 64] + [(47, 17), (48, 16), (55, 9)]
    out = []
    for _ in range(3):
        for w, total, rest in few:
            p = np.full(64, rest, dtype=np.uint32)
            n = np.full(w, total // w) + (np.arange(w) < total % w)
            for k, at in zip(n, rng.choice(64, size=w, replace=False)):
                p[at] = 0xFFFFFFFF & ~sum(1 << int(b) for b in rng.choice(32, size=k, replace=False))
            out.append(p)
        for n, o in half:
            p = np.zeros(64, dtype=np.uint32)
            at = rng.permutation(64)
            for a in at[:n]:
                p[a] = sum(1 << int(b) for b in rng.choice(32, size=16, replace=False))
            p[at[n:n + o]] = 0xFFFFFFFF
            out.append(p)
    return np.stack(out)


# the last number of rows of one size of logits and the first of the next: 8, 64, 256 and 384 MB
@pytest.mark.parametrize("dtype,B", [("bf16", 27), ("bf16", 28), ("bf16", 220), ("bf16", 221), ("bf16", 883), ("bf16", 884), ("bf16", 1325), ("bf16", 1326),
                                     ("f32", 13), ("f32", 14), ("f32", 110), ("f32", 111), ("f32", 441), ("f32", 442), ("f32", 662), ("f32", 663)])
def test_pieces_around_the_lines(xg, dtype, B):
    import torch
    dev = torch.device("cuda:0")
    V, rng = 151936, np.random.default_rng(B)                       # (rows of whole 128-byte lines: words 64 k .. 64 k + 63 are a piece)
    W = V // 32
    pieces = torch.from_numpy(_pieces(rng).view(np.int32)).to(dev)
    n = (W + 63) // 64
    which = torch.from_numpy((np.arange(B * n) + rng.integers(len(pieces))).reshape(B, n) % len(pieces)).to(dev)
    bm = pieces[which].reshape(B, n * 64)[:, :W].contiguous()
    tt, ninf = (torch.int16, -128) if dtype == "bf16" else (torch.int32, -8388608)     # 0xFF80, 0xFF800000
    logits = torch.randint(-2 ** 15, 2 ** 15, (B, V), generator=torch.Generator(device=dev).manual_seed(B), device=dev, dtype=tt)
    want = torch.empty_like(logits)
    for b in range(0, B, 128):
        allowed = ((bm[b:b + 128, :, None] >> torch.arange(32, device=dev, dtype=torch.int32)) & 1).view(-1, V).bool()
        want[b:b + 128] = torch.where(allowed, logits[b:b + 128], torch.tensor(ninf, device=dev, dtype=tt))
    xg.apply_token_bitmask(logits.data_ptr(), xg.XG2_BF16 if dtype == "bf16" else xg.XG2_F32, B, V, V, bm.data_ptr(), W,
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(logits, want)
