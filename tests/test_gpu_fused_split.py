"""The fused quantizer + linear on both sides of its kernels' lines (split reduction on 16 or 32 rows a workgroup, weight
resident from 4096 rows), in the three forms: the same bits as the two-launch form, whose kernels have their own tests."""
import pytest
import torch

import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
bits = lambda t: t.view(torch.int16)


@pytest.mark.parametrize("B,L,K,N,pad", [
    (21, 98, 64, 1, 0), (13, 163, 448, 128, 3), (16, 255, 1536, 80, 0),   # at most one workgroup of 16 rows per CU
    (17, 241, 320, 97, 0), (101, 197, 768, 56, 8),                       # few resident rows a CU
    (21, 195, 256, 72, 0), (32, 128, 256, 72, 4),                        # the line between split and resident
    (83, 57, 384, 128, 0), (61, 89, 1024, 40, 0), (42, 197, 576, 64, 0),  # 8-row units: 2, 4 and 1 k-steps in flight
    (104, 197, 320, 80, 0), (104, 199, 192, 33, 1), (211, 98, 1088, 16, 0),  # resident: odd step counts, ragged rows
])
def test_fused_forms_aligned(B, L, K, N, pad):
    print(f"fused split B={B} L={L} K={K} N={N}", flush=True)
    c = synth.random_problem(9100 + K + N, B, L, K, N, device=DEV)
    M = B * L
    wq, s_w, inv_m = ptq.fold_smoothing(c.w, c.m)
    xq, acc, acc2 = (torch.empty((M, n), dtype=t, device=DEV) for n, t in ((K, torch.int8), (N, torch.int32), (N, torch.int32)))
    buf = torch.full((M, N + pad), 777.0, dtype=torch.float16, device=DEV)

    q = ptq.quantize_pts(c.x, inv_m, c.s_tok, B, L)
    y = ptq.w8a8_linear(q, wq, c.s_tok, s_w, c.bias, B, L, acc_out=acc)
    ptq.w8a8_linear_fused(c.x, inv_m, c.s_tok, wq, s_w, c.bias, B, L, y=buf[:, :N])
    assert torch.equal(bits(buf[:, :N].contiguous()), bits(y)) and bool((buf[:, N:] == 777.0).all())
    y2 = ptq.w8a8_linear_fused(c.x, inv_m, c.s_tok, wq, s_w, c.bias, B, L, acc_out=acc2, xq_out=xq)
    assert torch.equal(bits(y2), bits(y)) and torch.equal(acc2, acc) and torch.equal(xq, q)

    z = torch.randint(-128, 128, (L,), dtype=torch.int32, device=DEV)
    rowsum = ptq.weight_rowsum(wq)
    q = ptq.quantize_pts_offset(c.x, inv_m, c.s_tok, z, B, L)
    y = ptq.w8a8_linear_offset(q, wq, c.s_tok, z, rowsum, s_w, None, B, L, acc_out=acc)
    y2 = ptq.w8a8_linear_offset_fused(c.x, inv_m, c.s_tok, z, wq, rowsum, s_w, None, B, L, acc_out=acc2, xq_out=xq)
    assert torch.equal(bits(y2), bits(y)) and torch.equal(acc2, acc) and torch.equal(xq, q)

    s4 = (c.s_tok * (127.0 / 7.0)).contiguous()
    wq4, s_w4, _ = ptq.fold_smoothing_w4(c.w, c.m)
    q4 = ptq.quantize_pts_a4(c.x, None, s4, B, L)
    y = ptq.w4a4_linear(q4, wq4, s4, s_w4, c.bias, B, L, acc_out=acc)
    y2 = ptq.w4a4_linear_fused(c.x, None, s4, wq4, s_w4, c.bias, B, L, acc_out=acc2, xq_out=xq)
    assert torch.equal(bits(y2), bits(y)) and torch.equal(acc2, acc)
    codes = torch.stack((((q4.int() << 28) >> 28), ((q4.int() << 24) >> 28)), 2).view(M, K).to(torch.int8)
    assert torch.equal(xq, codes)


@pytest.mark.parametrize("B,L,K,N", [(1, 17, 5, 3), (3, 65, 200, 130), (5, 197, 333, 1000), (16, 211, 1001, 127), (30, 199, 72, 96)])
def test_fused_w8a8_any_alignment(B, L, K, N):
    print(f"fused split unaligned B={B} L={L} K={K} N={N}", flush=True)
    c = synth.random_problem(9300 + K + N, B, L, K, N, device=DEV)
    wq, s_w, inv_m = ptq.fold_smoothing(c.w, c.m)
    q = ptq.quantize_pts(c.x, inv_m, c.s_tok, B, L)
    acc, acc2 = (torch.empty((B * L, N), dtype=torch.int32, device=DEV) for _ in range(2))
    y = ptq.w8a8_linear(q, wq, c.s_tok, s_w, c.bias, B, L, acc_out=acc)
    xq = torch.empty_like(q)
    y2 = ptq.w8a8_linear_fused(c.x, inv_m, c.s_tok, wq, s_w, c.bias, B, L, acc_out=acc2, xq_out=xq)
    y3 = ptq.w8a8_linear_fused(c.x, inv_m, c.s_tok, wq, s_w, c.bias, B, L)
    assert torch.equal(bits(y2), bits(y)) and torch.equal(bits(y3), bits(y)) and torch.equal(acc2, acc) and torch.equal(xq, q)
