"""Host-only checks of the Python callables: what they refuse before anything reaches the library.  The tensors are fake (a
CUDA device, a shape and no storage), so a call whose arguments pass gets as far as the launch and fails there."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import build as hip_build

B, L, K, N = 3, 4, 64, 40
M = B * L
H, F, I8, U8, I32 = torch.float16, torch.float32, torch.int8, torch.uint8, torch.int32


@pytest.fixture(scope="module", autouse=True)
def built():
    import os

    if not (os.path.exists(ptq.binding.LIB_PATH) and os.path.exists(ptq.binding.CALLS_PATH)):
        hip_build.build()


def fake(dtype, *shape):
    with FakeTensorMode(allow_non_fake_inputs=True):
        return torch.empty(shape, dtype=dtype, device="cuda:0")


def calls():
    """name: (arguments in order, {output argument: (dtype, rows, columns that are written)})"""
    x, inv_m, s_tok, z = fake(H, M, K), fake(F, K), fake(F, L), fake(I32, L)
    xq, wq, s_w, rs, bias = fake(I8, M, K), fake(I8, N, K), fake(F, N), fake(I32, N), fake(H, N)
    x4, w4, w16 = fake(U8, M, K // 2), fake(U8, N, K // 2), fake(H, N, K)
    x6, w6 = fake(U8, 1, M, 96), fake(U8, 1, N, 96)
    y = {"y": (H, M, N)}
    return {
        "quantize_pts": ((x, inv_m, s_tok, B, L), {"xq": (I8, M, K)}),
        "quantize_dynamic": ((x, inv_m), {"xq": (I8, M, K)}),
        "quantize_pts_offset": ((x, inv_m, s_tok, z, B, L), {"xq": (I8, M, K)}),
        "quantize_pts_a4": ((x, inv_m, s_tok, B, L), {"xq4": (U8, M, K // 2)}),
        "w8a8_linear": ((xq, wq, s_tok, s_w, bias, B, L), y),
        "w8a8_linear_offset": ((xq, wq, s_tok, z, rs, s_w, bias, B, L), y),
        "w4a4_linear": ((x4, w4, s_tok, s_w, bias, B, L), y),
        "w4a4_linear_e2m3": ((x6, w6, s_tok, s_w, bias, B, L, K), y),
        "w8a8_linear_fused": ((x, inv_m, s_tok, wq, s_w, bias, B, L), y),
        "w8a8_linear_offset_fused": ((x, inv_m, s_tok, z, wq, rs, s_w, bias, B, L), y),
        "w4a4_linear_fused": ((x, inv_m, s_tok, w4, s_w, bias, B, L), y),
        "f16_linear": ((x, w16, bias), y),
        # offline preparation
        "fold_smoothing": ((w16, inv_m), {"wq": (I8, N, K)}),
        "fold_smoothing_w4": ((w16, inv_m), {"wq4": (U8, N, K // 2)}),
    }


@pytest.mark.parametrize("name", calls())
def test_outputs_that_are_too_small_are_refused(name):
    args, outputs = calls()[name]
    for key, (dtype, rows, cols) in outputs.items():
        for shape in ((1, cols), (rows - 1, cols), (rows, cols - 1), (0, cols)):
            with pytest.raises(ValueError, match=f"{key}: expected at least {rows} x {cols}"):
                getattr(ptq, name)(*args, **{key: fake(dtype, *shape)})


@pytest.mark.parametrize("name", calls())
def test_outputs_of_the_right_size_or_larger_pass(name):
    args, outputs = calls()[name]
    for key, (dtype, rows, cols) in outputs.items():
        for shape in ((rows, cols), (rows + 5, cols), (rows, cols + 8)):
            with pytest.raises(RuntimeError):  # the launch: no device here, no storage anywhere
                getattr(ptq, name)(*args, **{key: fake(dtype, *shape)})


@pytest.mark.parametrize("name", [n for n in calls() if not n.startswith("fold")])
def test_wrong_types_and_arguments_are_refused(name):
    args, outputs = calls()[name]
    call = getattr(ptq, name)
    for key, (dtype, rows, cols) in outputs.items():
        with pytest.raises(TypeError, match=key):
            call(*args, **{key: fake(F, rows, cols)})
        with pytest.raises(TypeError, match=key):  # inner stride
            call(*args, **{key: fake(dtype, cols, rows).t()})
    with pytest.raises(TypeError, match="unexpected keyword argument 'nothing'"):
        call(*args, nothing=1)
    with pytest.raises(TypeError, match="missing required argument"):
        call(*args[:-1])
    with pytest.raises(TypeError):
        call(args[0].float(), *args[1:])


@pytest.mark.parametrize("name", [n for n in calls() if not n.startswith("fold") and n not in ("quantize_dynamic", "f16_linear")])
@pytest.mark.parametrize("b,l", [(B + 1, L), (1 << 62, 4), ((1 << 62) + B, L), (-(1 << 62), 8)])
def test_batch_times_tokens_is_exact(name, b, l):
    """B * L has to be the number of rows, also where the product leaves 64 bits."""
    args, _ = calls()[name]
    at = next(i for i, a in enumerate(args) if isinstance(a, int))
    args = list(args)
    args[at:at + 2] = [b, l]
    if l != L:  # the token vectors have l entries, and the activations as many rows as the wrapped product
        rows = (b * l + (1 << 63)) % (1 << 64) - (1 << 63)
        args = [fake(a.dtype, l) if isinstance(a, torch.Tensor) and tuple(a.shape) == (L,) else a for a in args]
        args[0] = fake(args[0].dtype, *(rows if d == M else d for d in args[0].shape))
    with pytest.raises(ValueError):
        getattr(ptq, name)(*args)


class _NoMemory(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is torch.ops.aten.empty.memory_format:
            raise torch.OutOfMemoryError("no room")
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("name", [n for n in calls() if not n.startswith("fold")])
def test_an_output_that_does_not_fit_raises_torchs_exception(name):
    args, _ = calls()[name]
    with _NoMemory(), pytest.raises(torch.OutOfMemoryError, match="no room"):
        getattr(ptq, name)(*args)


@pytest.mark.gpu
def test_an_output_larger_than_the_device():
    x = torch.zeros((1 << 21, 8), dtype=torch.float16, device="cuda:0")
    with pytest.raises(torch.OutOfMemoryError):  # 8 TiB of y
        ptq.f16_linear(x, x, None)
    with pytest.raises(torch.OutOfMemoryError):
        ptq.w8a8_linear(x.char(), x.char(), torch.ones(1 << 21, device="cuda:0"), torch.ones(1 << 21, device="cuda:0"), None, 1, 1 << 21)
