"""Thin binding of libptq4vm.so: argument marshalling only.

Every function takes torch CUDA tensors (used purely as device buffers), passes raw device
pointers, sizes and the current HIP stream to the C ABI declared in include/ptq4vm.h, and
returns the output tensors.  No arithmetic happens here and there is no fallback: if the
library has not been built, loading raises.

The launches of the hot path (quantizers and linears) are callables of the extension module
_calls (host/calls.cc), which does the same checks natively; the offline preparation of weights
and the validator go through ctypes here.
"""
from __future__ import annotations

import ctypes
import importlib
import os
import sys
import sysconfig
from typing import Optional, Tuple

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# PTQ4VM_LIB: another build of the same sources (the sanitized host build of the test suite)
LIB_PATH = os.environ.get("PTQ4VM_LIB") or os.path.join(_HERE, "libptq4vm.so")
CALLS_PATH = os.path.join(_HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

EXPORTS = (
    "ptq4vm_fold_smoothing",
    "ptq4vm_quantize_pts",
    "ptq4vm_quantize_dynamic",
    "ptq4vm_quantize_pts_offset",
    "ptq4vm_weight_rowsum",
    "ptq4vm_w8a8_linear_offset",
    "ptq4vm_fold_smoothing_w4",
    "ptq4vm_quantize_pts_a4",
    "ptq4vm_w4a4_linear",
    "ptq4vm_fold_smoothing_w4_e2m3",
    "ptq4vm_quantize_pts_a4_e2m3",
    "ptq4vm_w4a4_linear_e2m3",
    "ptq4vm_w4a4_linear_fused",
    "ptq4vm_w8a8_linear_offset_fused",
    "ptq4vm_w8a8_linear",
    "ptq4vm_w8a8_linear_fused",
    "ptq4vm_f16_linear",
    "ptq4vm_validate_scales",
    "ptq4vm_validate_scales_static",
    "ptq4vm_status_string",
    "ptq4vm_last_hip_error",
    "ptq4vm_version",
)

_lib = None


class Ptq4vmError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"ptq4vm status {status}: {text}")
        self.status = status


def load() -> ctypes.CDLL:
    """Load libptq4vm.so (built by paper_2412_20386_amd.build). Raises if it is missing."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(
            f"{LIB_PATH} not found: " + _BUILD_HINT)
    lib = ctypes.CDLL(LIB_PATH)
    i64, vp, ci = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
    lib.ptq4vm_fold_smoothing.restype = ci
    lib.ptq4vm_fold_smoothing.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, vp]
    lib.ptq4vm_quantize_pts.restype = ci
    lib.ptq4vm_quantize_pts.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_quantize_dynamic.restype = ci
    lib.ptq4vm_quantize_dynamic.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, vp]
    lib.ptq4vm_quantize_pts_offset.restype = ci
    lib.ptq4vm_quantize_pts_offset.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_weight_rowsum.restype = ci
    lib.ptq4vm_weight_rowsum.argtypes = [vp, vp, i64, i64, i64, vp]
    lib.ptq4vm_w8a8_linear_offset.restype = ci
    lib.ptq4vm_w8a8_linear_offset.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_fold_smoothing_w4.restype = ci
    lib.ptq4vm_fold_smoothing_w4.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, vp]
    lib.ptq4vm_quantize_pts_a4.restype = ci
    lib.ptq4vm_quantize_pts_a4.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_w4a4_linear.restype = ci
    lib.ptq4vm_w4a4_linear.argtypes = [vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_fold_smoothing_w4_e2m3.restype = ci
    lib.ptq4vm_fold_smoothing_w4_e2m3.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i64, vp]
    lib.ptq4vm_quantize_pts_a4_e2m3.restype = ci
    lib.ptq4vm_quantize_pts_a4_e2m3.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_w4a4_linear_e2m3.restype = ci
    lib.ptq4vm_w4a4_linear_e2m3.argtypes = [vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_w8a8_linear_offset_fused.restype = ci
    lib.ptq4vm_w8a8_linear_offset_fused.argtypes = [vp] * 11 + [i64] * 8 + [vp]
    lib.ptq4vm_w4a4_linear_fused.restype = ci
    lib.ptq4vm_w4a4_linear_fused.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_w8a8_linear.restype = ci
    lib.ptq4vm_w8a8_linear.argtypes = [vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_w8a8_linear_fused.restype = ci
    lib.ptq4vm_w8a8_linear_fused.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, i64,
                                             i64, vp]
    lib.ptq4vm_f16_linear.restype = ci
    lib.ptq4vm_f16_linear.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, i64, vp]
    lib.ptq4vm_validate_scales.restype = ci
    lib.ptq4vm_validate_scales.argtypes = [vp, i64, vp, i64, vp, i64, vp, vp, i64, vp]
    lib.ptq4vm_validate_scales_static.restype = ci
    lib.ptq4vm_validate_scales_static.argtypes = [vp, i64, vp, i64, vp, i64, vp, vp]
    lib.ptq4vm_status_string.restype = ctypes.c_char_p
    lib.ptq4vm_status_string.argtypes = [ci]
    lib.ptq4vm_last_hip_error.restype = ctypes.c_char_p
    lib.ptq4vm_last_hip_error.argtypes = []
    lib.ptq4vm_version.restype = ci
    lib.ptq4vm_version.argtypes = []
    _lib = lib
    return lib


# ---------------------------------------------------------------------------------- launches of the hot path
HOT_CALLS = ("quantize_pts", "quantize_dynamic", "quantize_pts_offset", "quantize_pts_a4", "quantize_pts_a4_e2m3",
             "w8a8_linear", "w8a8_linear_offset", "w4a4_linear", "w4a4_linear_e2m3", "w8a8_linear_fused",
             "w8a8_linear_offset_fused", "w4a4_linear_fused", "f16_linear")


def _load_entries() -> None:
    """Hand the library's entry points to _calls (its callables ask for this on their first call)."""
    lib = load()
    _calls.bind({name: ctypes.cast(getattr(lib, "ptq4vm_" + name), ctypes.c_void_p).value for name in HOT_CALLS})


_BUILD_HINT = "build it with `python -m paper_2412_20386_amd.build` (there is no CPU or PyTorch fallback)"


def _bind_calls() -> None:
    """Import the extension and put its callables in the place of the stand-ins, here and in the package."""
    if not os.path.exists(CALLS_PATH):
        raise FileNotFoundError(f"{CALLS_PATH} not found: " + _BUILD_HINT)
    importlib.invalidate_caches()  # (it may have been built a moment ago)
    try:
        from . import _calls as extension

        callables = {name: getattr(extension, name) for name in HOT_CALLS}
    except (ImportError, AttributeError) as err:  # built for another torch or Python, or from other sources
        raise ImportError(f"{CALLS_PATH} does not fit this package ({err}): " + _BUILD_HINT) from err
    extension.setup(_load_entries, check)
    globals()["_calls"] = extension
    for namespace in (globals(), vars(sys.modules[__package__])):
        namespace.update({name: call for name, call in callables.items() if namespace.get(name, _stand_ins[name]) is _stand_ins[name]})


def _stand_in(name: str):
    """A callable that binds the extension when it is first called: importing the package needs no built extension, and the
    package builds it."""
    def call(*args, **kwargs):
        if globals()[name] is call:
            _bind_calls()
        return globals()[name](*args, **kwargs)
    call.__name__ = name
    return call


_stand_ins = {_name: _stand_in(_name) for _name in HOT_CALLS}


def status_string(status: int) -> str:
    return load().ptq4vm_status_string(int(status)).decode()


def check(status: int) -> None:
    if status != 0:
        text = status_string(status)
        if status == -5:
            text += ": " + load().ptq4vm_last_hip_error().decode()
        raise Ptq4vmError(status, text)


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()  # plain ints: the declared argtypes convert them


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _matrix(t: torch.Tensor, dtype, name: str) -> Tuple[int, int, int]:
    if not t.is_cuda or t.dtype != dtype or t.dim() != 2 or (t.shape[1] > 1 and t.stride(1) != 1):
        raise TypeError(f"{name}: expected a 2-D CUDA tensor of {dtype} with unit inner stride")
    return t.shape[0], t.shape[1], (t.stride(0) if t.shape[0] > 1 else max(t.stride(0), t.shape[1]))


def _written(t: torch.Tensor, dtype, rows: int, cols: int, name: str) -> int:
    """Pitch of a matrix that the library writes rows x cols elements of.  A larger one is taken too; the C boundary sees a
    pointer and a pitch only, so a smaller one has to be refused here."""
    r, c, ld = _matrix(t, dtype, name)
    if r < rows or c < cols:
        raise ValueError(f"{name}: expected at least {rows} x {cols} elements, got {r} x {c}")
    return ld


def _vector(t: Optional[torch.Tensor], dtype, n: int, name: str, optional=False):
    if t is None:
        if optional:
            return
        raise TypeError(f"{name} is required")
    if not t.is_cuda or t.dtype != dtype or t.dim() != 1 or t.shape[0] != n or not t.is_contiguous():
        raise TypeError(f"{name}: expected a contiguous CUDA vector of {n} x {dtype}")


def fold_smoothing(w: torch.Tensor, m: torch.Tensor, wq: Optional[torch.Tensor] = None):
    """ptq4vm_fold_smoothing: (wq int8 [N,K], s_w f32 [N], inv_m f32 [K])."""
    N, K, ldw = _matrix(w, torch.float16, "w")
    _vector(m, torch.float32, K, "m")
    if wq is None:
        wq = torch.empty((N, K), dtype=torch.int8, device=w.device)
    ldwq = _written(wq, torch.int8, N, K, "wq")
    s_w = torch.empty(N, dtype=torch.float32, device=w.device)
    inv_m = torch.empty(K, dtype=torch.float32, device=w.device)
    check(load().ptq4vm_fold_smoothing(_ptr(w), _ptr(m), _ptr(wq), _ptr(s_w), _ptr(inv_m), N, K, ldw, ldwq,
                                       _stream()))
    return wq, s_w, inv_m


def weight_rowsum(wq: torch.Tensor) -> torch.Tensor:
    """ptq4vm_weight_rowsum: int32 [N] = sum_k wq[o, k]."""
    N, K, ldwq = _matrix(wq, torch.int8, "wq")
    out = torch.empty(N, dtype=torch.int32, device=wq.device)
    check(load().ptq4vm_weight_rowsum(_ptr(wq), _ptr(out), N, K, ldwq, _stream()))
    return out


def fold_smoothing_w4(w: torch.Tensor, m: torch.Tensor, wq4: Optional[torch.Tensor] = None):
    """ptq4vm_fold_smoothing_w4: (wq4 uint8 [N, K/2] packed, s_w f32 [N], inv_m f32 [K])."""
    N, K, ldw = _matrix(w, torch.float16, "w")
    _vector(m, torch.float32, K, "m")
    if wq4 is None:
        wq4 = torch.empty((N, K // 2), dtype=torch.uint8, device=w.device)
    ldwq = _written(wq4, torch.uint8, N, K // 2, "wq4")
    s_w = torch.empty(N, dtype=torch.float32, device=w.device)
    inv_m = torch.empty(K, dtype=torch.float32, device=w.device)
    check(load().ptq4vm_fold_smoothing_w4(_ptr(w), _ptr(m), _ptr(wq4), _ptr(s_w), _ptr(inv_m), N, K, ldw, ldwq,
                                          _stream()))
    return wq4, s_w, inv_m


def e2m3_blocks(K: int) -> int:
    """PTQ4VM_E2M3_BLOCKS: 96-byte blocks of 128 codes that a row of K codes takes in the E2M3 container."""
    return (K + 127) // 128


def _e2m3_container(t: torch.Tensor, rows: int, K: int, what: str) -> int:
    """Checks a block-major container [e2m3_blocks(K), rows, 96] uint8 and returns its plane pitch in bytes."""
    if not isinstance(t, torch.Tensor) or not t.is_cuda or t.dtype != torch.uint8 or t.dim() != 3:
        raise TypeError(f"{what}: expected a CUDA uint8 tensor [blocks, rows, 96]")
    if tuple(t.shape) != (e2m3_blocks(K), rows, 96) or t.stride(2) != 1 or (rows > 1 and t.stride(1) != 96):
        raise ValueError(f"{what}: expected shape {(e2m3_blocks(K), rows, 96)} with dense 96-byte blocks")
    return t.stride(0) if t.shape[0] > 1 else max(t.stride(0), 96 * rows)


def fold_smoothing_w4_e2m3(w: torch.Tensor, m: torch.Tensor, wq6: Optional[torch.Tensor] = None):
    """ptq4vm_fold_smoothing_w4_e2m3: (wq6 uint8 [e2m3_blocks(K), N, 96] block-major, s_w f32 [N], inv_m f32 [K])."""
    N, K, ldw = _matrix(w, torch.float16, "w")
    _vector(m, torch.float32, K, "m")
    if wq6 is None:
        wq6 = torch.empty((e2m3_blocks(K), N, 96), dtype=torch.uint8, device=w.device)
    ldwq = _e2m3_container(wq6, N, K, "wq6")
    s_w = torch.empty(N, dtype=torch.float32, device=w.device)
    inv_m = torch.empty(K, dtype=torch.float32, device=w.device)
    check(load().ptq4vm_fold_smoothing_w4_e2m3(_ptr(w), _ptr(m), _ptr(wq6), _ptr(s_w), _ptr(inv_m), N, K, ldw, ldwq,
                                               _stream()))
    return wq6, s_w, inv_m


VALIDATE_BLOCK = 4096  # PTQ4VM_VALIDATE_BLOCK


def validate_scales(s_tok: Optional[torch.Tensor], m: Optional[torch.Tensor], s_w: Optional[torch.Tensor],
                    workspace: Optional[torch.Tensor] = None) -> Tuple[int, torch.Tensor]:
    """ptq4vm_validate_scales: (status, bad_counts int32 [3] on the device).  status is 0 or
    PTQ4VM_ERR_VALUE (-6, some entry is not a finite number > 0); other errors raise.  Synchronises."""
    vecs = [v for v in (s_tok, m, s_w) if v is not None]
    if not vecs:
        raise TypeError("at least one vector is required")
    dev = vecs[0].device
    sizes = []
    for v, name in ((s_tok, "s_tok"), (m, "m"), (s_w, "s_w")):
        if v is not None:
            _vector(v, torch.float32, v.shape[0], name)
        sizes.append(0 if v is None else v.shape[0])
    need = 16 * ((sum(sizes) + VALIDATE_BLOCK - 1) // VALIDATE_BLOCK + 1)
    if workspace is None:
        workspace = torch.empty(need, dtype=torch.uint8, device=dev)
    counts = torch.empty(3, dtype=torch.int32, device=dev)
    rc = load().ptq4vm_validate_scales(_ptr(s_tok), sizes[0], _ptr(m), sizes[1], _ptr(s_w), sizes[2], _ptr(counts),
                                       _ptr(workspace), workspace.numel() * workspace.element_size(), _stream())
    if rc not in (0, -6):
        check(rc)
    return rc, counts


def validate_scales_static(s_tok: Optional[torch.Tensor], m: Optional[torch.Tensor], s_w: Optional[torch.Tensor],
                           counts: torch.Tensor) -> None:
    """ptq4vm_validate_scales_static: enqueue only; `counts` (int32 [3], device, the caller's) holds the bad-entry
    counts once the current stream has run the two kernels.  Allocates nothing and does not synchronise."""
    sizes = []
    for v, name in ((s_tok, "s_tok"), (m, "m"), (s_w, "s_w")):
        if v is not None:
            _vector(v, torch.float32, v.shape[0], name)
        sizes.append(0 if v is None else v.shape[0])
    _vector(counts, torch.int32, 3, "counts")
    check(load().ptq4vm_validate_scales_static(_ptr(s_tok), sizes[0], _ptr(m), sizes[1], _ptr(s_w), sizes[2],
                                               _ptr(counts), _stream()))


globals().update(_stand_ins)
try:
    _bind_calls()
except (FileNotFoundError, ImportError):
    pass  # raised again, with the reason, by the first call
