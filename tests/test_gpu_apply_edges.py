"""Masking of logits wherever the rows begin and end relative to the vectors, cache lines and pieces that the kernel works in,
and with logits too large for the last-level cache.  Bit for bit; what surrounds the rows is untouched.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _stream():
    import torch
    return torch.cuda.current_stream().cuda_stream


@pytest.fixture(scope="module")
def xg():
    import torch
    assert torch.cuda.is_available()
    import paper_2601_04426_amd as xg
    return xg


# V: within a vector, a mask word, a piece of 2,048 tokens, a workgroup's 8,192 and around them; pad: row strides of any residue
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 3, 8, 31, 33, 63, 64, 65, 1000, 1985, 2047, 2048, 2049, 8129, 8192, 8193, 50021])
def test_rows_at_any_place(xg, dtype, V):
    import torch
    dev = torch.device("cuda:0")
    u, i, code = (np.uint32, np.int32, xg.XG2_F32) if dtype == "f32" else (np.uint16, np.int16, xg.XG2_BF16)
    size = np.dtype(u).itemsize
    rng = np.random.default_rng(V)
    B, W = 5, (V + 31) // 32
    allow = np.stack([rng.random(V) < d for d in (0.0, 1.0, 0.5, 0.01, 0.99)])
    bm = np.stack([oracle.pack_bitmask(a) for a in allow])
    bm_t = torch.from_numpy(bm).to(dev)
    # offsets in bytes: every place in a vector, around a line, and (last) off a multiple of the element
    offsets = [size * k for k in range(16 // size)] + [112, 128 - size, 128, 128 + size, size // 2]
    for off in offsets:
        for pad in (0, 1, 5, 64):
            stride = V + pad
            n = B * stride
            raw = rng.integers(0, 256, size=256 + n * size + 256, dtype=np.uint8)
            t = torch.from_numpy(raw).to(dev)
            assert t.data_ptr() % 256 == 0
            xg.apply_token_bitmask(t.data_ptr() + 128 + off, code, B, V, stride, bm_t.data_ptr(), W, _stream())
            torch.cuda.synchronize()
            want = raw.copy()
            rows = np.frombuffer(want[128 + off:128 + off + n * size].tobytes(), dtype=u).reshape(B, stride).copy()
            part = np.ascontiguousarray(rows[:, :V])
            (oracle.apply_f32 if dtype == "f32" else oracle.apply_bf16)(part, bm)
            rows[:, :V] = part
            want[128 + off:128 + off + n * size] = np.frombuffer(rows.tobytes(), dtype=np.uint8)
            assert np.array_equal(t.cpu().numpy(), want), (off, pad)


@pytest.mark.parametrize("dtype,B,V", [("bf16", 883, 152001), ("bf16", 884, 152001), ("f32", 447, 150001), ("f32", 448, 150001)])
def test_large_logits(xg, dtype, B, V):
    """Just below and above 2^28 bytes, where streaming stores take over."""
    import torch
    dev = torch.device("cuda:0")
    W = (V + 31) // 32
    tt = torch.int16 if dtype == "bf16" else torch.int32
    ninf = -128 if dtype == "bf16" else -8388608                      # 0xFF80, 0xFF800000
    g = torch.Generator(device=dev).manual_seed(B)
    logits = torch.randint(-2 ** 15, 2 ** 15, (B, V), generator=g, device=dev, dtype=tt)
    words = torch.randint(-2 ** 31, 2 ** 31, (B, W), generator=g, device=dev, dtype=torch.int64)
    words[::3] = -1
    words[1::3] &= words[1::3].roll(1, 1) & words[1::3].roll(2, 1) & words[1::3].roll(3, 1)
    bm = words.to(torch.int32)
    want = logits.clone()
    tok = torch.arange(V, device=dev)
    for b in range(B):
        allowed = (bm[b][tok >> 5] >> (tok & 31).to(torch.int32)) & 1
        want[b][allowed == 0] = ninf
    xg.apply_token_bitmask(logits.data_ptr(), xg.XG2_BF16 if dtype == "bf16" else xg.XG2_F32, B, V, V, bm.data_ptr(), W, _stream())
    torch.cuda.synchronize()
    assert torch.equal(logits, want)
