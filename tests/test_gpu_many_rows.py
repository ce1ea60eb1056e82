"""Row counts at which one workgroup per small tile would be 2^32 threads or more, the limit of a grid dimension: the tile
kernels and the split reduction of the fused form; and the longest sequence of the quantizers.  Steps are powers of two, so
outputs are exact."""
import pytest
import torch

import paper_2412_20386_amd as ptq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 1 << 27


def _rows(lo, hi):
    return torch.arange(lo, hi, dtype=torch.int32, device=DEV) if hi < 2 ** 31 else torch.arange(lo, hi, device=DEV)


def test_f16_linear_beyond_a_billion_rows():
    M = (1 << 30) + 13
    print(f"f16 M={M} K=1 N=1", flush=True)
    x = torch.empty((M, 1), dtype=torch.float16, device=DEV)
    for lo in range(0, M, CHUNK):
        hi = min(M, lo + CHUNK)
        x[lo:hi, 0] = (_rows(lo, hi) % 2039).half()
    y = ptq.f16_linear(x, torch.full((1, 1), 0.5, dtype=torch.float16, device=DEV), None)
    for lo in range(0, M, CHUNK):
        hi = min(M, lo + CHUNK)
        assert torch.equal(y[lo:hi], x[lo:hi] * 0.5), lo


def test_w8a8_linears_beyond_two_billion_rows():
    L, B = 7, 306783379
    M = B * L
    assert M > 2 ** 31
    print(f"w8a8 and fused M={M} K=1 N=1", flush=True)
    x = torch.empty((M, 1), dtype=torch.float16, device=DEV)
    for lo in range(0, M, CHUNK):
        hi = min(M, lo + CHUNK)
        x[lo:hi, 0] = (_rows(lo, hi) % 253 - 126).half()
    s_tok = torch.tensor([2.0 ** -t for t in range(L)], device=DEV)
    one, w = torch.ones(1, device=DEV), torch.full((1, 1), 3, dtype=torch.int8, device=DEV)
    xq = ptq.quantize_pts(x, None, torch.ones(L, device=DEV), B, L)
    y = ptq.w8a8_linear(xq, w, s_tok, one, None, B, L)
    for lo in range(0, M, CHUNK):
        hi = min(M, lo + CHUNK)
        t = (_rows(lo, hi) % L).long()
        assert torch.equal(xq[lo:hi], x[lo:hi].to(torch.int8)), lo
        assert torch.equal(y[lo:hi, 0], (x[lo:hi, 0].float() * 3 * s_tok[t]).half()), lo
    y.zero_()
    ptq.w8a8_linear_fused(x, None, torch.ones(L, device=DEV), w, one, None, B, L, y=y)
    for lo in range(0, M, CHUNK):
        hi = min(M, lo + CHUNK)
        assert torch.equal(y[lo:hi], x[lo:hi] * 3), lo


def test_quantizers_longest_sequence():
    """L = 2^31 - 1: the token position that follows a thread's last row lies beyond 2^31."""
    L, K = 2 ** 31 - 1, 8
    print(f"quantizers L={L} K={K}", flush=True)
    x = torch.empty((L, K), dtype=torch.float16, device=DEV)
    for lo in range(0, L, CHUNK):
        hi = min(L, lo + CHUNK)
        x[lo:hi] = (_rows(lo, hi) % 127 - 63).half()[:, None]
    s_tok = torch.ones(L, device=DEV)
    s_tok[1::2] = 0.5
    for quantize, dtype in ((ptq.quantize_pts, torch.int8), (ptq.quantize_pts_a4, torch.uint8)):
        q = quantize(x, None, s_tok, 1, L)
        for lo in range(0, L, CHUNK):
            hi = min(L, lo + CHUNK)
            want = (_rows(lo, hi) % 127 - 63) * (1 + _rows(lo, hi) % 2)
            if dtype is torch.uint8:
                want = want.clamp(-7, 7) & 15
                want = want | (want << 4)
            assert bool((q[lo:hi] == want.to(dtype)[:, None]).all()), lo
        del q
