"""Which kernel a call runs on, by its name in the profiler's record, on both sides of the lines of the dispatch, with the
result checked against a 64-bit product.  The shapes are the smallest that reach a kernel, ragged in rows and channels."""
import warnings

import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2412_20386_amd as ptq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PERSISTENT, STREAM, SMALLK = "linear_mfma_persistent<", "linear_stream_smallk<", "linear_mfma_smallk<"
TILE, SPLITK, WRES, SPLIT, FUSED_TILE = "linear_mfma_tile<", "linear_mfma_splitk<", "pts_linear_wres<", "pts_linear_split<", "pts_linear_generic<"
E_PERSISTENT, E_TILE, E_SPLITK = "linear_e2m3_persistent<", "linear_e2m3_tile<", "linear_e2m3_splitk<"
DIRECT, STAGED, ONE_SLAB = "Copy)0>", "Copy)1>", "Copy)2>"  # how linear_mfma_tile brings its slabs


def ran(call):
    """Names of this library's kernels that the call launched."""
    call()
    torch.cuda.synchronize()
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        with profile(activities=[ProfilerActivity.CUDA]) as record:
            call()
            torch.cuda.synchronize()
    return [e.key for e in record.key_averages() if "linear" in e.key and "<" in e.key]


def check_kernel(call, *parts):
    names = ran(call)
    assert len(names) == 1 and all(p in names[0] for p in parts), (names, parts)


def rows_of(L, M):
    return torch.arange(M, device=DEV) % L


def close(y, acc64, scale, bias):
    """One fp16 rounding plus the fp32 roundings of the epilogue."""
    p = acc64 * scale
    y64 = p if bias is None else p + bias.double()
    tol = 2.0 ** -10 * y64.abs() + 2.0 ** -21 * (p.abs() + (0 if bias is None else bias.double().abs())) + 2.0 ** -24
    return bool(((y.double() - y64).abs() <= tol).all())


class Problem:
    def __init__(self, M, K, N, L=None, limit=127):
        g = torch.Generator(device=DEV).manual_seed(M + 3 * K + 7 * N)
        ints = lambda lo, hi, *s: torch.randint(lo, hi, s, generator=g, device=DEV)
        self.L = L = L or next(d for d in (11, 7, 5, 3, 2, 1) if M % d == 0)
        self.M, self.K, self.N, self.B = M, K, N, M // L
        self.x, self.w = ints(-limit, limit + 1, M, K).to(torch.int8), ints(-limit, limit + 1, N, K).to(torch.int8)
        self.s_tok, self.s_w = (torch.rand(n, generator=g, device=DEV) * 0.01 + 0.001 for n in (L, N))
        self.bias = torch.randn(N, generator=g, device=DEV).half()
        self.z = ints(-128, 128, L).to(torch.int32)
        self.rowsum = self.w.sum(1, dtype=torch.int32)
        self.acc64 = self.x.double() @ self.w.double().t()
        self.scale = self.s_tok.double()[rows_of(L, M)][:, None] * self.s_w.double()[None, :]
        self.acc = torch.empty((M, N), dtype=torch.int32, device=DEV)


@pytest.mark.parametrize("M,K,N", [
    (128 * 2303 + 5, 384, 256), (128 * 191 + 77, 384, 3072), (128 * 575 + 1, 768, 1024), (128 * 767 + 100, 768, 768),
])
def test_persistent_kernel_over_many_tiles(M, K, N):
    """Short reductions over whole rounds of 128 x 256 units; ragged last tiles; one column of tiles and several, full and
    half tiles; with and without bias; with the accumulators; and one row unit less."""
    print(f"persistent M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N)
    for bias in (p.bias, None):
        run = lambda **kw: ptq.w8a8_linear(p.x, p.w, p.s_tok, p.s_w, bias, p.B, p.L, **kw)
        check_kernel(run, PERSISTENT, "Int8Path")
        y = run()
        assert close(y, p.acc64, p.scale, bias)
        check_kernel(lambda: run(acc_out=p.acc), PERSISTENT)
        p.acc.fill_(-1)
        y_dump = run(acc_out=p.acc)
        assert torch.equal(p.acc.double(), p.acc64) and torch.equal(y_dump.view(torch.int16), y.view(torch.int16))
    M = (M // 128) * 128 - M // 128 // 100
    x = p.x[:M]
    check_kernel(lambda: ptq.w8a8_linear(x, p.w, p.s_tok[:1], p.s_w, p.bias, M, 1), PERSISTENT)


def _e2m3(p):
    x6 = ptq.quantize_pts_a4_e2m3(p.x.half(), None, torch.ones(p.L, device=DEV), p.B, p.L)
    p.w[:, 0] = 7  # every weight row folds to step 1
    w6, step, _ = ptq.fold_smoothing_w4_e2m3(p.w.half(), torch.ones(p.K, device=DEV))
    assert bool((step == 1).all())
    p.acc64 = p.x.double() @ p.w.double().t()
    return x6, w6


@pytest.mark.parametrize("M,K,N,kernel", [
    (31301, 256, 1032, E_PERSISTENT), (17451, 384, 2056, E_PERSISTENT),      # 615 and 621 tiles, 8 channels in the last; 2 and 3 blocks
    (31232, 256, 1032, E_TILE), (26373, 256, 1032, E_TILE), (14807, 384, 2056, E_TILE), (26112, 256, 1032, E_TILE),  # 610, 520, 522 and 510 tiles
    (12301, 256, 1024, E_PERSISTENT), (12288, 256, 1024, E_TILE),             # 776 and 768 tiles of 128 x 128
    (13312, 384, 1024, E_TILE), (13312, 1152, 1024, E_PERSISTENT),            # 832: from there long reductions only
    (17000, 1152, 1032, E_TILE), (26900, 384, 520, E_TILE),                   # more than one round; padding
])
def test_e2m3_kernels(M, K, N, kernel):
    """The persistent kernel down to its shortest reduction (fewer blocks than ring stages), ragged in rows and channels, with
    and without bias, with the accumulators; and what lies just beyond its lines."""
    print(f"e2m3 M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N, limit=7)
    x6, w6 = _e2m3(p)
    for bias in (p.bias, None):
        run = lambda **kw: ptq.w4a4_linear_e2m3(x6, w6, p.s_tok, p.s_w, bias, p.B, p.L, p.K, **kw)
        check_kernel(run, kernel)
        y = run()
        assert close(y, p.acc64, p.scale, bias)
        p.acc.fill_(-1)
        check_kernel(lambda: run(acc_out=p.acc), kernel)
        assert torch.equal(p.acc.double(), p.acc64)
        assert torch.equal(run(acc_out=p.acc).view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("M,K,N,kernel", [
    (20480, 66, 160, TILE), (20483, 68, 160, TILE), (20479, 68, 160, TILE), (20501, 100, 416, TILE), (20501, 100, 424, TILE),
    (27999, 72, 128, TILE), (28001, 72, 128, TILE), (39999, 72, 96, TILE), (40003, 72, 96, TILE),
    (36001, 76, 132, TILE), (36001, 76, 130, TILE), (35999, 76, 132, TILE), (36001, 76, 196, TILE),
    (29999, 128, 416, TILE), (30001, 128, 416, TILE), (20483, 128, 448, TILE), (20483, 128, 2080, TILE),  # 65 to 128 codes
    (32768, 24, 768, STREAM), (32767, 24, 768, TILE), (32768, 24, 776, TILE), (32768, 26, 768, TILE), (32768, 64, 768, TILE),  # 24 M results in whole lines
    (98304, 12, 256, STREAM), (20479, 48, 1536, TILE), (20483, 48, 1536, STREAM), (20483, 16, 1600, STREAM), (20483, 16, 1728, TILE),  # (no more channels fit the LDS)
])
def test_short_reductions_over_many_rows(M, K, N, kernel):
    """In the three forms (packed 4-bit: the same number of codes, so half the bytes and half the alignment)."""
    print(f"stream M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N)
    check_kernel(lambda: ptq.w8a8_linear(p.x, p.w, p.s_tok, p.s_w, p.bias, p.B, p.L), kernel)
    y = ptq.w8a8_linear(p.x, p.w, p.s_tok, p.s_w, p.bias, p.B, p.L, acc_out=p.acc)
    assert close(y, p.acc64, p.scale, p.bias) and torch.equal(p.acc.double(), p.acc64)
    offset = lambda: ptq.w8a8_linear_offset(p.x, p.w, p.s_tok, p.z, p.rowsum, p.s_w, None, p.B, p.L, acc_out=p.acc)
    check_kernel(offset, kernel)
    z = p.z.double()[rows_of(p.L, M)][:, None] * p.rowsum.double()[None, :]
    assert close(offset(), p.acc64 - z, p.scale, None) and torch.equal(p.acc.double(), p.acc64)
    x4, w4 = p.x.clamp(-7, 7), p.w.clamp(-7, 7)
    pack = lambda c: ((c[:, 0::2] & 15) | ((c[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous()
    xp, wp = pack(x4), pack(w4)
    packed = lambda: ptq.w4a4_linear(xp, wp, p.s_tok, p.s_w, p.bias, p.B, p.L, acc_out=p.acc)
    check_kernel(packed, TILE if K // 2 % 4 else STREAM if K == 64 else kernel)  # (64 packed codes are no whole step of bytes)
    acc4 = x4.double() @ w4.double().t()
    assert close(packed(), acc4, p.scale, p.bias) and torch.equal(p.acc.double(), acc4)


@pytest.mark.parametrize("M,K,N,more,kernel", [
    (32768, 24, 768, 0, SMALLK), (32767, 24, 768, 0, TILE), (32771, 24, 776, 0, TILE), (32771, 24, 768, 2, SMALLK), (32771, 26, 768, 0, TILE),
    (32771, 24, 768, 1, TILE), (32771, 32, 768, 0, TILE), (32771, 8, 768, 0, SMALLK), (16391, 48, 1536, 0, SMALLK), (16391, 56, 1600, 0, SMALLK),
    (16391, 40, 1536, 8, SMALLK), (200003, 17, 128, 3, SMALLK), (200003, 64, 128, 8, TILE),
])
def test_f16_short_reductions(M, K, N, more, kernel):
    """Channel strips from 24 M results in whole lines, if rows start at 16-byte boundaries (up to 24 elements at 4-byte ones).  Infinities
    beyond K stay out; without and with bias."""
    print(f"f16 short M={M} K={K} N={N} more={more}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + K + N)
    x, w = (torch.full((r, K + more), float("inf"), dtype=torch.float16, device=DEV)[:, :K] for r in (M, N))
    x.copy_(torch.randn(M, K, generator=g, device=DEV))
    w.copy_(torch.randn(N, K, generator=g, device=DEV))
    y64, mag = x.double() @ w.double().t(), x.double().abs() @ w.double().abs().t()
    for bias in (None, torch.randn(N, generator=g, device=DEV).half()):
        check_kernel(lambda: ptq.f16_linear(x, w, bias), kernel)
        want = y64 if bias is None else y64 + bias.double()
        assert bool(((ptq.f16_linear(x, w, bias).double() - want).abs() <= (K + 2) * 2.0 ** -24 * (mag + 4.0) + 2.0 ** -10 * want.abs() + 2.0 ** -24).all())


@pytest.mark.parametrize("M,K,N,parts", [
    (16 * 16, 1536, 16 * 16, (SPLITK,)), (16 * 16 + 1, 64, 16 * 16, (TILE, "32, 64", DIRECT)),
    (1001, 960, 832, (TILE, "64, 64", DIRECT)), (3137, 448, 1153, (TILE, "64, 128", DIRECT)), (6209, 192, 1025, (TILE, "128, 128", DIRECT)),
    (13057, 192, 2048, (TILE, "128, 256", DIRECT)), (65536, 256, 256, (PERSISTENT,)), (65536, 256, 416, (PERSISTENT,)), (65536, 256, 408, (TILE, "128, 256")), (65281, 256, 264, (TILE,)),
    # any pitch and K: one slab (63, 64 unaligned rows, 128), two with one byte in the second, more; each tile
    (12345, 63, 2179, (TILE, "128, 128", ONE_SLAB)), (12345, 65, 2179, (TILE, "128, 128", STAGED)), (6401, 1030, 900, (TILE, "128, 128", "128, 2,", STAGED)),
    (6401, 63, 1029, (TILE, "64, 128", ONE_SLAB)), (6401, 65, 1029, (TILE, "64, 128", STAGED)), (1279, 33, 645, (TILE, "64, 64", ONE_SLAB)),
    (1279, 129, 645, (TILE, "64, 64", STAGED)), (2049, 321, 643, (TILE, "64, 64", "128, 2,", STAGED)), (401, 127, 899, (TILE, "32, 64", ONE_SLAB)),
    (401, 130, 899, (TILE, "32, 64", STAGED)), (46670, 250, 61, (TILE, "64, 64", STAGED)), (401, 1001, 403, (SPLITK, "2, 2")), (50, 13, 7, (SPLITK, "1, 1")),
])
def test_int8_tiles(M, K, N, parts):
    print(f"tiles M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N)
    run = lambda **kw: ptq.w8a8_linear(p.x, p.w, p.s_tok, p.s_w, p.bias, p.B, p.L, **kw)
    check_kernel(run, *parts)
    y = run()
    assert close(y, p.acc64, p.scale, p.bias)
    p.acc.fill_(-1)
    run(acc_out=p.acc)
    assert torch.equal(p.acc.double(), p.acc64)


@pytest.mark.parametrize("M,K,N,parts", [
    (25009, 448, 380, (TILE, "256, 192", DIRECT)), (25009, 320, 380, (TILE, "128, 128", DIRECT)),  # from 384 bytes of K
    (22785, 384, 384, (TILE, "256, 192", DIRECT)), (22784, 384, 384, (TILE, "128, 128", DIRECT)),  # 180 and 178 of 256
    (8705, 320, 1536, (TILE, "256, 256", DIRECT)), (8704, 320, 1536, (TILE, "128, 128", DIRECT)),  # 210 and 204 of 256
    (4225, 64, 520, (TILE, "64, 64", "128, 3,", DIRECT)), (50001, 192, 56, (TILE, "64, 64", "128, 2,", DIRECT)),  # 603 and 782 tiles
])
def test_int8_tiles_of_whole_rounds(M, K, N, parts):
    test_int8_tiles(M, K, N, parts)


@pytest.mark.parametrize("M,K,N,parts", [
    (49153, 448, 384, (TILE, "256, 192", DIRECT)), (48897, 448, 384, (TILE, "256, 192", DIRECT)), (48896, 448, 384, (TILE, "128, 128", DIRECT)),  # 386, 384 and 382 of 512
    (65536, 448, 384, (TILE, "256, 192", DIRECT)), (65537, 448, 384, (TILE, "128, 128", DIRECT)),  # 512 and 514 of 768
    (23274, 832, 1024, (TILE, "128, 128", DIRECT)), (24577, 448, 1500, (TILE, "128, 256", DIRECT)),  # 546 and 776
])
def test_int8_tiles_of_a_few_rounds(M, K, N, parts):
    """256 x 192 tiles: one round filled to 70 %, two to 75 %, never three."""
    test_int8_tiles(M, K, N, parts)


@pytest.mark.parametrize("kind,M,K,N,parts", [
    ("packed", 13057, 384, 2048, ("Int4Path", "128, 256, 2, 4, 64, 3", DIRECT)), ("f16", 13057, 96, 2048, ("Half16Path", "128, 256, 2, 4, 64, 3", DIRECT)),
    ("offset", 13057, 192, 2048, ("Int8OffsetPath", "128, 256, 2, 4, 64, 3", DIRECT)), ("packed", 13057, 384, 2045, ("Int4Path", "128, 256", DIRECT)),
    ("packed", 49153, 384, 56, ("Int4Path", "64, 64, 2, 2, 128, 2", DIRECT)), ("f16", 49153, 96, 56, ("Half16Path", "64, 64, 2, 2, 128, 2", DIRECT)),
    ("offset", 49153, 192, 56, ("Int8OffsetPath", "64, 64, 2, 2, 128, 2", DIRECT)), ("offset", 32769, 320, 50, ("Int8OffsetPath", "64, 64, 2, 2, 128, 2", DIRECT)),
    ("offset", 25009, 448, 380, ("Int8OffsetPath", "256, 192", DIRECT)), ("f16", 25009, 224, 380, ("Half16Path", "256, 192", DIRECT)),
    ("packed", 25009, 896, 380, ("Int4Path", "128, 128", DIRECT)),  # (never on 256-row tiles)
    ("offset", 8705, 320, 1536, ("Int8OffsetPath", "256, 256", DIRECT)), ("f16", 8705, 160, 1536, ("Half16Path", "256, 256", DIRECT)),
])
def test_direct_tiles_of_the_other_operands(kind, M, K, N, parts):
    """The largest tiles, the tiles of whole rounds and the two-stage 64 x 64 tiles on each of the other operand types."""
    print(f"{kind} tiles M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N, limit=7 if kind == "packed" else 127)
    if kind == "f16":
        x, w = p.x.half() / 64, p.w.half() / 64  # (exact; products sum without rounding)
        run = lambda **kw: ptq.f16_linear(x, w, p.bias)
        check_kernel(run, TILE, *parts)
        assert close(run(), p.acc64 / 4096, torch.ones((), dtype=torch.float64, device=DEV), p.bias)
        return
    if kind == "packed":
        pack = lambda c: ((c[:, 0::2] & 15) | ((c[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous()
        x, w = pack(p.x), pack(p.w)
        run = lambda **kw: ptq.w4a4_linear(x, w, p.s_tok, p.s_w, p.bias, p.B, p.L, **kw)
        want = p.acc64
    else:
        run = lambda **kw: ptq.w8a8_linear_offset(p.x, p.w, p.s_tok, p.z, p.rowsum, p.s_w, p.bias, p.B, p.L, **kw)
        want = p.acc64 - p.z.double()[rows_of(p.L, M)][:, None] * p.rowsum.double()[None, :]
    check_kernel(run, TILE, *parts)
    y = run()
    assert close(y, want, p.scale, p.bias)
    p.acc.fill_(-1)
    assert torch.equal(run(acc_out=p.acc).view(torch.int16), y.view(torch.int16)) and torch.equal(p.acc.double(), p.acc64)


@pytest.mark.parametrize("M,K,N,more,parts", [
    (800, 513, 320, 0, (SPLITK, "2, 2")), (801, 513, 320, 0, (TILE, "32, 64", STAGED)),  # 250 and 260 blocks
    (800, 512, 320, 2, (SPLITK, "2, 2")), (801, 514, 320, 0, (TILE, "32, 64", STAGED)),
    (3200, 516, 320, 0, (SPLITK, "2, 2")), (3201, 516, 320, 0, (TILE, "64, 64", STAGED)), (3200, 512, 320, 4, (SPLITK, "2, 2")),  # 1000 and 1010
])
def test_split_and_staged_by_the_rows(M, K, N, more, parts):
    test_one_slab_by_the_rows(M, K, N, more, parts)


FRAGMENTS, VIA_LDS = "false, (ptq4vm::mfma::Copy)2>", "true, (ptq4vm::mfma::Copy)2>"


@pytest.mark.parametrize("M,K,N,more,parts", [
    (12345, 60, 2179, 0, (TILE, "128, 128", FRAGMENTS)), (12345, 61, 2179, 0, (TILE, "128, 128", VIA_LDS)), (12345, 64, 2179, 2, (TILE, "128, 128", VIA_LDS)),
    (6401, 63, 1029, 1, (TILE, "64, 128", FRAGMENTS)), (6401, 64, 1029, 1, (TILE, "64, 128", VIA_LDS)),
    (1279, 12, 645, 0, (TILE, "64, 64", FRAGMENTS)), (1279, 12, 645, 3, (TILE, "64, 64", VIA_LDS)),
    (401, 64, 899, 1, (TILE, "32, 64", FRAGMENTS)), (401, 65, 899, 0, (TILE, "32, 64", VIA_LDS)), (401, 128, 899, 4, (TILE, "32, 64", FRAGMENTS)),
])
def test_one_slab_by_the_rows(M, K, N, more, parts):
    """Rows at multiples of 4 bytes (and the smallest tiles up to 64 bytes) as fragments, others through LDS; the operands' rows are part
    of wider ones."""
    print(f"one slab M={M} K={K} N={N} more={more}", flush=True)
    p = Problem(M, K, N)
    wide = lambda t: torch.nn.functional.pad(t, (0, more), value=127)[:, :K]
    x, w = wide(p.x), wide(p.w)
    run = lambda **kw: ptq.w8a8_linear(x, w, p.s_tok, p.s_w, p.bias, p.B, p.L, **kw)
    check_kernel(run, *parts)
    y = run(acc_out=p.acc)
    assert close(y, p.acc64, p.scale, p.bias) and torch.equal(p.acc.double(), p.acc64)
    assert torch.equal(run().view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("M,K,N,parts", [
    (32769, 256, 56, (TILE, "64, 64", "128, 2,", DIRECT)), (32768, 256, 56, (TILE, "64, 64", "128, 3,", DIRECT)),  # 513 and 512 tiles
    (49152, 192, 56, (TILE, "64, 64", "128, 3,", DIRECT)), (49153, 192, 56, (TILE, "64, 64", "128, 2,", DIRECT)),  # 768 and 769
])
def test_stages_of_the_64_x_64_tiles(M, K, N, parts):
    """Two ring stages instead of three from 513 tiles on, from 769 where K is shorter than 256 bytes."""
    test_int8_tiles(M, K, N, parts)


@pytest.mark.parametrize("M,K,N", [(12345, 31, 2179), (12345, 33, 2179), (5121, 520, 900), (6401, 32, 1028), (6401, 33, 1029), (401, 66, 899), (2049, 200, 643)])
def test_f16_tiles_any_alignment(M, K, N):
    """fp32 accumulation in any order, |error| <= (K + 2) 2^-24 sum |terms|, and one fp16 rounding.  Infinities beyond K (the
    padding of wider rows) stay out."""
    print(f"f16 tiles M={M} K={K} N={N}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + K + N)
    x, w = (torch.full((r, K + 1 + K % 2), float("inf"), dtype=torch.float16, device=DEV)[:, :K] for r in (M, N))  # odd pitch
    x.copy_(torch.randn(M, K, generator=g, device=DEV))
    w.copy_(torch.randn(N, K, generator=g, device=DEV))
    check_kernel(lambda: ptq.f16_linear(x, w, None), TILE)
    y, y64, mag = ptq.f16_linear(x, w, None), x.double() @ w.double().t(), x.double().abs() @ w.double().abs().t()
    assert bool(((y.double() - y64).abs() <= (K + 2) * 2.0 ** -24 * mag + 2.0 ** -10 * y64.abs() + 2.0 ** -24).all())


@pytest.mark.parametrize("M,K,N,parts", [
    (2048, 256, 72, (SPLIT, "1, 8")), (4095, 1536, 80, (SPLIT, "1, 8")), (4096, 1536, 80, (WRES, "<5,")), (4099, 192, 33, (WRES, "<3,")),
    (7167, 1280, 92, (WRES, "<6,", "false, true>")), (7168, 1280, 92, (WRES, "<6,", "false, false>")), (7167, 704, 92, (WRES, "<6,", "false, false>")),
    (33001, 256, 113, (WRES, "<8,")), (50001, 384, 100, (WRES, "<7,")), (40003, 832, 90, (WRES, "<6,")),
    (4096, 100, 300, (STREAM,)), (1000, 100, 300, (SPLIT,)), (5000, 200, 128, (SPLIT, "2, 4")), (2048, 200, 130, (SPLIT,)), (2049, 200, 130, (FUSED_TILE,)),
])
def test_fused_kernels(M, K, N, parts):
    """The one-launch form: the codes, accumulators and outputs of the two-launch form."""
    print(f"fused M={M} K={K} N={N}", flush=True)
    p = Problem(M, K, N)
    x = (torch.randn(M, K, generator=torch.Generator(device=DEV).manual_seed(K), device=DEV) * 0.3).half()
    inv_m = torch.rand(K, device=DEV) + 0.5
    run = lambda **kw: ptq.w8a8_linear_fused(x, inv_m, p.s_tok, p.w, p.s_w, p.bias, p.B, p.L, **kw)
    check_kernel(run, *parts)
    q = ptq.quantize_pts(x, inv_m, p.s_tok, p.B, p.L)
    y = ptq.w8a8_linear(q, p.w, p.s_tok, p.s_w, p.bias, p.B, p.L)
    acc64 = q.double() @ p.w.double().t()
    assert close(run(), acc64, p.scale, p.bias)
    codes = torch.empty_like(q)
    y_dump = run(acc_out=p.acc, xq_out=codes)
    assert torch.equal(codes, q) and torch.equal(p.acc.double(), acc64)
    assert torch.equal(run().view(torch.int16), y.view(torch.int16)) and torch.equal(y_dump.view(torch.int16), y.view(torch.int16))
