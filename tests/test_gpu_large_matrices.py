"""Reductions that end inside a step, over activations of more than 2 GiB: the last pieces of a row are put right by their distance from
the matrix's end, which no longer fits 32 bits there.  int32 accumulators against fp32 products that are exact (K 127^2 < 2^24)."""
import pytest
import torch

import paper_2412_20386_amd as ptq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 1 << 20


def same(acc, x, w):
    wt = w.float().t().contiguous()
    for lo in range(0, acc.shape[0], CHUNK):
        hi = min(lo + CHUNK, acc.shape[0])
        assert torch.equal(acc[lo:hi], (x[lo:hi].float() @ wt).int()), lo


def codes(R, K, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randint(-127, 128, (R, K), generator=g, device=DEV, dtype=torch.int8)


def scales(M, N):
    return torch.ones(1, device=DEV), torch.ones(N, device=DEV) * 2.0 ** -10, torch.empty((M, N), dtype=torch.int32, device=DEV)


@pytest.mark.parametrize("K,N", [(129, 8), (33, 8), (3, 5)])  # staged tiles, one slab, a weight under 16 bytes
def test_linear(K, N):
    M = (2 << 30) // K + 70007
    print(f"M={M} K={K} N={N}", flush=True)
    x, w = codes(M, K, 1), codes(N, K, 2)
    s_tok, s_w, acc = scales(M, N)
    ptq.w8a8_linear(x, w, s_tok, s_w, None, M, 1, acc_out=acc)
    same(acc, x, w)


def test_split_reduction_over_long_rows():
    M, K, N, pitch = 300, 101, 40, (1 << 23) + 5  # (pitches beyond what a tile's 32-bit offsets reach)
    print(f"M={M} K={K} N={N} pitch={pitch}", flush=True)
    x, w = torch.empty(M * pitch, dtype=torch.int8, device=DEV).view(M, pitch)[:, :K], codes(N, K, 2)
    x.copy_(codes(M, K, 1))
    s_tok, s_w, acc = scales(M, N)
    ptq.w8a8_linear(x, w, s_tok, s_w, None, M, 1, acc_out=acc)
    same(acc, x, w)


def test_fused_linear():
    K, N = 67, 8
    M = (2 << 30) // (2 * K) + 70007
    print(f"fused M={M} K={K} N={N}", flush=True)
    q, w = codes(M, K, 1), codes(N, K, 2)
    s_tok, s_w, acc = scales(M, N)
    ptq.w8a8_linear_fused(q.half(), None, s_tok, w, s_w, None, M, 1, acc_out=acc)
    same(acc, q, w)
