"""The linears' kernels at the edges of their tiles (csrc/gemm_tile.hpp, csrc/gemm_e2m3.hip), on every operand type, against a 64-bit
product (exact for the integer paths).  A shape's comment names the tiles of the 8-bit linear unless it says otherwise; which kernel a
shape runs on is asserted in test_gpu_routes.py."""
import pytest
import torch

import paper_2412_20386_amd as ptq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [  # M, K, N (int8 reductions; every operand type picks its own tile from the same rule), pitch of y beyond N
    (1, 64, 1, 0), (33, 192, 17, 1), (255, 1536, 80, 0),           # split reduction over 16 x 16 blocks: one element, ragged, long
    (65, 128, 2049, 0), (197, 1088, 769, 3),                       # 32 x 64 tiles; K ends in half a slab; odd rows of y
    (785, 192, 1601, 0), (1001, 960, 832, 8),                      # 64 x 64 tiles, three ring stages
    (1999, 320, 1216, 0),                                          # 64 x 64 tiles, two ring stages (packed: three)
    (3137, 448, 1153, 0),                                          # 64 x 128 tiles
    (6209, 192, 1025, 5), (49217, 1536, 80, 0),                    # 128 x 128 tiles, and with a column tile mostly padding
    (13057, 192, 2048, 0),                                         # 128 x 256 tiles (fp16: persistent; packed: any alignment)
    (50, 13, 7, 0), (301, 100, 130, 0), (17, 1001, 333, 1),        # any alignment: 16 x 16 blocks
    (1111, 514, 402, 0), (1111, 516, 402, 0), (600, 514, 402, 0),  # 32 x 64 tiles; 32 x 32 blocks
    (401, 72, 899, 2), (1279, 200, 645, 0), (2049, 722, 643, 0),   # 32 x 64, 64 x 64 with short and long slabs
    (6401, 30, 1029, 0), (12345, 334, 2179, 1),                    # 64 x 128, 128 x 128
]


def _close(y, y64, magnitude):
    """One fp16 rounding (half an ulp, 2^-11 of the value; a whole ulp where fp32 rounding tips it) plus the fp32 roundings."""
    y = y.double()
    tol = 2.0 ** -10 * y64.abs() + 2.0 ** -21 * magnitude + 2.0 ** -24
    return bool(((y - y64).abs() <= tol).all())


def _output(M, N, pad):
    buf = torch.full((M, N + pad), 777.0, dtype=torch.float16, device=DEV)
    return buf, buf[:, :N]


@pytest.mark.parametrize("M,K,N,pad", SHAPES)
def test_tile_kernels_all_operand_types(M, K, N, pad):
    print(f"tiles M={M} K={K} N={N} pad={pad}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K + N)
    B, L = (M // 7, 7) if M % 7 == 0 else (1, M)
    ints = lambda lo, hi, *s: torch.randint(lo, hi, s, generator=g, device=DEV)
    xq, wq = ints(-127, 128, M, K).to(torch.int8), ints(-127, 128, N, K).to(torch.int8)
    s_tok = torch.rand(L, generator=g, device=DEV) * 0.01 + 0.001
    s_w = torch.rand(N, generator=g, device=DEV) * 0.01 + 0.001
    bias = torch.randn(N, generator=g, device=DEV).half()
    scale = s_tok.double().repeat(B)[:, None] * s_w.double()[None, :]

    def check(y, buf, acc64, sc, b):
        p = acc64 * sc
        assert _close(y, p + b.double(), p.abs() + b.double().abs())
        assert bool((buf[:, N:] == 777.0).all())

    # int8
    acc64 = xq.double() @ wq.double().t()
    acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
    buf, y = _output(M, N, pad)
    ptq.w8a8_linear(xq, wq, s_tok, s_w, bias, B, L, y=y)
    check(y, buf, acc64, scale, bias)
    y2 = ptq.w8a8_linear(xq, wq, s_tok, s_w, bias, B, L, acc_out=acc)
    assert torch.equal(acc.double(), acc64) and torch.equal(y2, y)

    # zero offset
    z = ints(-128, 128, L).to(torch.int32)
    rowsum = ptq.weight_rowsum(wq)
    buf, y = _output(M, N, pad)
    ptq.w8a8_linear_offset(xq, wq, s_tok, z, rowsum, s_w, bias, B, L, y=y)
    check(y, buf, acc64 - z.double().repeat(B)[:, None] * rowsum.double()[None, :], scale, bias)

    # packed 4-bit codes
    K2 = K - K % 2
    if K2:
        x4, w4 = ints(-7, 8, M, K2), ints(-7, 8, N, K2)
        pack = lambda c: ((c[:, 0::2] & 15) | ((c[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous()
        acc4 = x4.double() @ w4.double().t()
        buf, y = _output(M, N, pad)
        ptq.w4a4_linear(pack(x4), pack(w4), s_tok, s_w, bias, B, L, y=y, acc_out=acc)
        check(y, buf, acc4, scale, bias)
        assert torch.equal(acc.double(), acc4)

    # 4-bit codes in the E2M3 container: integer activations at step 1 are their own codes; an integer weight row whose
    # largest entry is 7 folds to step 1
    x4, w4 = ints(-7, 8, M, K), ints(-7, 8, N, K)
    w4[:, 0] = 7
    one = torch.ones(max(K, L), device=DEV)
    xq6 = ptq.quantize_pts_a4_e2m3(x4.half(), None, one[:L], B, L)
    wq6, step, _ = ptq.fold_smoothing_w4_e2m3(w4.half(), one[:K])
    assert bool((step == 1).all())
    acc4 = x4.double() @ w4.double().t()
    buf, y = _output(M, N, pad)
    ptq.w4a4_linear_e2m3(xq6, wq6, s_tok, s_w, bias, B, L, K, y=y, acc_out=acc)
    check(y, buf, acc4, scale, bias)
    assert torch.equal(acc.double(), acc4)

    # fp16, without and with bias: fp32 accumulation in any order, |error| <= (K + 2) 2^-24 sum |terms|
    x, w = torch.randn(M, K, generator=g, device=DEV).half(), torch.randn(N, K, generator=g, device=DEV).half()
    mag = x.double().abs() @ w.double().abs().t()
    for b in (None, bias):
        y64 = x.double() @ w.double().t() + (0 if b is None else b.double())
        buf, y = _output(M, N, pad)
        ptq.f16_linear(x, w, b, y=y)
        err = (y.double() - y64).abs()
        assert bool((err <= (K + 2) * 2.0 ** -24 * (mag + 4.0) + 2.0 ** -10 * y64.abs() + 2.0 ** -24).all())
        assert bool((buf[:, N:] == 777.0).all())


@pytest.mark.parametrize("M,K,N,pad", [
    (25009, 448, 380, 3),    # 256 x 192 tiles, K ends in half a slab, odd rows of y
    (25201, 1152, 376, 8),   # the same, whole slabs and 16-byte stores, the last tile partly empty both ways
    (9433, 320, 1531, 0),    # 256 x 256 tiles
    (40009, 128, 640, 0),    # E2M3: 128 x 256 tiles, results past the caches; integers: streamed; fp16: persistent
    (13057, 384, 2045, 3),   # packed: 128 x 256 tiles, the last 253 channels wide
    (13057, 96, 2048, 0),    # fp16: 128 x 256 tiles, results past the caches
    (12301, 64, 776, 0),     # 128 x 128 tiles of one step
    (97, 320, 2048, 0),      # more channels than rows: rows walked first
])
def test_tiles_of_whole_rounds(M, K, N, pad):
    """Tiles that take a CU each, the stores of large results, and the tile order of small ones."""
    test_tile_kernels_all_operand_types(M, K, N, pad)


@pytest.mark.parametrize("M,K,N,pad", [
    (33013, 256, 1016, 0),   # two blocks a tile, rows that are not whole lines, the last tile partly empty both ways
    (33013, 256, 1016, 8),   # the same with rows of whole lines
    (43777, 384, 768, 0),    # three blocks, a last tile of one row
    (39433, 256, 1016, 0), (39433, 256, 1016, 8), (52481, 384, 768, 0),  # the same for E2M3, whose rounds have to be filled
])
def test_persistent_tiles_with_stores_in_flight(M, K, N, pad):
    """Few blocks a tile: the copies of the next tile's first blocks, its scale vectors and this tile's stores in one queue."""
    test_tile_kernels_all_operand_types(M, K, N, pad)


@pytest.mark.parametrize("K,N,B,L", [(384, 3072, 124, 199), (768, 3072, 128, 197), (768, 1536, 190, 260)])
def test_persistent_kernel_against_smaller_launches(K, N, B, L):
    """Many rounds of tiles, with a part round in half tiles: the same bits as two launches of half the images, whose rounds and half
    tiles fall elsewhere."""
    print(f"persistent B={B} L={L} K={K} N={N}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(77 + K + N)
    M = B * L
    x = torch.randint(-127, 128, (M, K), dtype=torch.int8, device=DEV, generator=g)
    w = torch.randint(-127, 128, (N, K), dtype=torch.int8, device=DEV, generator=g)
    s_tok = torch.rand(L, device=DEV, generator=g) * 0.02 + 0.001
    s_w = torch.rand(N, device=DEV, generator=g) * 0.002 + 0.0001
    for bias in (None, torch.randn(N, device=DEV, generator=g).half()):
        y = ptq.w8a8_linear(x, w, s_tok, s_w, bias, B, L)
        half = M // 2
        parts = [ptq.w8a8_linear(p, w, s_tok, s_w, bias, B // 2, L) for p in (x[:half], x[half:])]
        assert torch.equal(torch.cat(parts).view(torch.int16), y.view(torch.int16))
