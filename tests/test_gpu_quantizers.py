"""The streaming quantizers at the edges of their chunks (8 elements), grids and token tables, in all forms, against the
oracle: rows that are no whole number of chunks, odd pitches, one row per thread and many."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
_np = lambda t: t.cpu().numpy()


def _view(rows, cols, pitch, dtype, fill):
    buf = torch.full((rows, pitch), fill, dtype=dtype, device=DEV)
    return buf, buf[:, :cols]


@pytest.mark.parametrize("B,L,K,pad_x,pad_q", [
    (1, 3, 6, 0, 0), (2, 5, 8, 0, 0), (3, 7, 9, 0, 1), (3, 7, 15, 1, 0), (2, 50, 16, 8, 8), (2, 33, 30, 2, 3),
    (2, 197, 128, 0, 0), (3, 65, 256, 0, 0), (2, 50, 1001, 0, 0), (40, 211, 1000, 0, 0), (30, 197, 502, 0, 0),
    (40, 197, 2048, 0, 0),  # more than four rows per thread: the table of reciprocal steps
    (90, 197, 1003, 0, 0),
])
def test_quantizer_forms_and_edges(B, L, K, pad_x, pad_q):
    print(f"quantizers B={B} L={L} K={K} pads {pad_x} {pad_q}", flush=True)
    c = synth.random_problem(8000 + B + L + K, B, L, K, 8, device=DEV)
    M = B * L
    _, x = _view(M, K, K + pad_x, torch.float16, 9.0)
    x.copy_(c.x)
    inv_m = (1.0 / c.m).contiguous()
    xn, mn, sn = _np(c.x), _np(inv_m), _np(c.s_tok)

    buf, q = _view(M, K, K + pad_q, torch.int8, 0x55)
    ptq.quantize_pts(x, inv_m, c.s_tok, B, L, xq=q)
    assert np.array_equal(_np(q), oracle.quantize_pts(xn, mn, sn, B, L)) and bool((buf[:, K:] == 0x55).all())

    z = torch.randint(-128, 128, (L,), dtype=torch.int32, device=DEV)
    buf, q = _view(M, K, K + pad_q, torch.int8, 0x55)
    ptq.quantize_pts_offset(x, inv_m, c.s_tok, z, B, L, xq=q)
    assert np.array_equal(_np(q), oracle.quantize_pts_offset(xn, mn, sn, _np(z), B, L)) and bool((buf[:, K:] == 0x55).all())

    buf, q = _view(M, K, K + pad_q, torch.int8, 0x55)
    _, s_row = ptq.quantize_dynamic(x, inv_m, xq=q)
    want, s_want = oracle.quantize_dynamic(xn, mn)
    assert np.array_equal(_np(q), want) and np.array_equal(_np(s_row), s_want) and bool((buf[:, K:] == 0x55).all())

    if K % 2 == 0:
        s4 = (c.s_tok * (127.0 / 7.0)).contiguous()
        buf, q = _view(M, K // 2, K // 2 + pad_q, torch.uint8, 0x55)
        ptq.quantize_pts_a4(x, inv_m, s4, B, L, xq4=q)
        want = oracle.pack_int4(oracle.quantize_pts_bits(xn, mn, _np(s4), B, L, 4))
        assert np.array_equal(_np(q), want) and bool((buf[:, K // 2:] == 0x55).all())
