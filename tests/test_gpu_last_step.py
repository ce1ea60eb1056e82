"""The last MFMA step of a reduction of any length and pitch: its 16-byte loads end at the matrix's last byte, what lies beyond K stays out, and a
matrix of fewer than 16 bytes has a kernel of its own.  The operands lie inside larger buffers whose other bytes would show
(infinities, codes of 127)."""
import pytest
import torch

import paper_2412_20386_amd as ptq
from test_gpu_routes import SPLIT, SPLITK, check_kernel, close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inside(values, pitch, fill):
    """`values` [R, K] as the rows of a buffer of `pitch` elements a row that ends with the last row's last element; everything
    around them is `fill`."""
    R, K = values.shape
    buf = torch.full((R * pitch + 64,), fill, dtype=values.dtype, device=DEV)
    view = buf[: R * pitch].view(R, pitch)[:, :K]
    view.copy_(values)
    return view


SHAPES = [  # M, K, N, elements that a row's pitch exceeds K by
    (1, 1, 1, 0), (1, 7, 3, 0), (1, 15, 200, 0), (3, 5, 40, 0), (15, 1, 17, 0), (700, 13, 1, 0), (5, 3, 1, 0),  # under 16 bytes
    (5003, 4, 3, 0), (700, 5, 2, 3), (9001, 1, 15, 0),                                                            # the weight alone
    (1, 16, 5, 0), (2, 8, 9, 0), (4, 5, 33, 1), (16, 1, 16, 0), (2, 9, 2, 7),                                   # 16 bytes and little more
    (1, 17, 3, 0), (33, 31, 49, 0), (65, 47, 130, 3), (7, 63, 20, 1), (40, 65, 24, 0), (17, 79, 33, 2),          # 16 x 16 blocks
    (90, 130, 300, 5), (33, 1648, 49, 0), (200, 257, 180, 0),
    (700, 300, 401, 0), (600, 515, 390, 0),                                                                       # 32 x 32 blocks
    (3000, 29, 700, 0), (3000, 63, 700, 1), (3000, 64, 700, 1), (401, 127, 899, 0), (401, 130, 899, 1),            # tiles, one slab and more
    (9000, 33, 1600, 0), (9000, 64, 1600, 2), (12345, 61, 2179, 0), (12345, 334, 2179, 1),
]


@pytest.mark.parametrize("M,K,N,more", SHAPES)
def test_last_step_of_the_linears(M, K, N, more):
    print(f"last step M={M} K={K} N={N} more={more}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + 5 * K + 11 * N)
    ints = lambda lo, hi, *s: torch.randint(lo, hi, s, generator=g, device=DEV)
    B, L = (M // 5, 5) if M % 5 == 0 else (1, M)
    s_tok, s_w = (torch.rand(n, generator=g, device=DEV) * 0.01 + 0.001 for n in (L, N))
    bias, acc = torch.randn(N, generator=g, device=DEV).half(), torch.empty((M, N), dtype=torch.int32, device=DEV)
    scale = s_tok.double().repeat(B)[:, None] * s_w.double()[None, :]

    x, w = (inside(ints(-127, 128, r, K).to(torch.int8), K + more, 127) for r in (M, N))
    acc64 = x.double() @ w.double().t()
    y = ptq.w8a8_linear(x, w, s_tok, s_w, bias, B, L, acc_out=acc)
    assert torch.equal(acc.double(), acc64) and close(y, acc64, scale, bias)
    z, rowsum = ints(-128, 128, L).to(torch.int32), w.sum(1, dtype=torch.int32)
    y = ptq.w8a8_linear_offset(x, w, s_tok, z, rowsum, s_w, bias, B, L)
    assert close(y, acc64 - z.double().repeat(B)[:, None] * rowsum.double()[None, :], scale, bias)

    packed = [ints(0, 256, r, K).to(torch.uint8) for r in (M, N)]  # 2 K codes a row
    signed = lambda n: (n.double() + 8) % 16 - 8
    codes = [torch.stack((signed(p & 15), signed(p >> 4)), 2).view(p.shape[0], 2 * K) for p in packed]
    acc4 = codes[0] @ codes[1].t()
    y = ptq.w4a4_linear(inside(packed[0], K + more, 0x77), inside(packed[1], K + more, 0x77), s_tok, s_w, bias, B, L, acc_out=acc)
    assert torch.equal(acc.double(), acc4) and close(y, acc4, scale, bias)

    inf = float("inf")
    x, w = (inside(torch.randn(r, K, generator=g, device=DEV).half(), K + more, inf) for r in (M, N))
    y, y64, mag = ptq.f16_linear(x, w, bias), x.double() @ w.double().t() + bias.double(), x.double().abs() @ w.double().abs().t()
    assert bool(((y.double() - y64).abs() <= (K + 2) * 2.0 ** -24 * (mag + 4.0) + 2.0 ** -10 * y64.abs() + 2.0 ** -24).all())


@pytest.mark.parametrize("M,K,N,more", [s for s in SHAPES if s[2] <= 128 or s[0] <= 2048] + [(5001, 71, 57, 1), (9000, 7, 2, 0)])
def test_last_step_of_the_fused_linear(M, K, N, more):
    """The codes, accumulators and outputs of the two-launch form."""
    print(f"last step, fused M={M} K={K} N={N} more={more}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + 5 * K + 11 * N)
    B, L = (M // 5, 5) if M % 5 == 0 else (1, M)
    s_tok, s_w = (torch.rand(n, generator=g, device=DEV) * 0.01 + 0.001 for n in (L, N))
    w = inside(torch.randint(-127, 128, (N, K), generator=g, device=DEV).to(torch.int8), K + more, 127)
    x = inside((torch.randn(M, K, generator=g, device=DEV) * 0.3).half(), K + more, float("nan"))
    for inv_m in (None, torch.rand(K, generator=g, device=DEV) + 0.5):
        codes, acc = torch.empty((M, K), dtype=torch.int8, device=DEV), torch.empty((M, N), dtype=torch.int32, device=DEV)
        y = ptq.w8a8_linear_fused(x, inv_m, s_tok, w, s_w, None, B, L, acc_out=acc, xq_out=codes)
        q = ptq.quantize_pts(x, inv_m, s_tok, B, L)
        assert torch.equal(codes, q) and torch.equal(acc.double(), q.double() @ w.double().t())
        assert torch.equal(y.view(torch.int16), ptq.w8a8_linear(q, w, s_tok, s_w, None, B, L).view(torch.int16))


@pytest.mark.parametrize("M,K,N,tiny", [(1, 15, 200, True), (1, 16, 200, False), (5, 3, 1, True), (16, 1, 16, False), (700, 13, 1, True), (700, 13, 2, False)])
def test_matrices_under_16_bytes(M, K, N, tiny):
    x, w = torch.ones((M, K), dtype=torch.int8, device=DEV), torch.ones((N, K), dtype=torch.int8, device=DEV)
    s_tok, s_w = torch.ones(1, device=DEV), torch.ones(N, device=DEV)
    check_kernel(lambda: ptq.w8a8_linear(x, w, s_tok, s_w, None, M, 1), SPLITK, "1, 1, 1, 1, " if tiny else "1, 1, 4, 4, ")
    tiny = min(2 * M, N) * K < 16  # (fp16 activations)
    check_kernel(lambda: ptq.w8a8_linear_fused(x.half(), None, s_tok, w, s_w, None, M, 1), SPLIT, "1, 1, 1, " if tiny else "1, 8, ")
