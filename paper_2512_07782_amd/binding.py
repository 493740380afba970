"""Python binding with the same names as the C ABI (include/gfwa.h).

Each function takes torch tensors living on the GPU, checks shapes/dtypes/contiguity on the
host, and passes raw device pointers and the current HIP stream to the library.  There is no
fallback: if `libgfwa.so` has not been built the import of the library raises.

The calls of the method itself go through a native module (`_gfwa_call`, csrc/binding.cpp), which does the
checks and allocates the outputs that were not given; the size queries, calibration and instrumentation
calls go through ctypes.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os
from typing import Optional, Tuple

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# GFWA_LIB names another build of the same library (a host-sanitizer build, for one)
_LIB_PATH = os.environ.get("GFWA_LIB") or os.path.join(_HERE, "libgfwa.so")
_CALL_PATH = os.path.join(_HERE, "_gfwa_call.so")
_lib: Optional[ctypes.CDLL] = None
_call = None  # the native module, bound to _lib's functions
# the functions it calls, in the order its bind() expects them
_CALLED = ("gfwa_gate_prefix", "gfwa_gate_activation_prefix", "gfwa_gate_activation_backward",
           "gfwa_gate_scan_workspace_bytes", "gfwa_gate_prefix_stp", "gfwa_forward_gqa", "gfwa_backward_workspace_bytes",
           "gfwa_backward_gqa", "gfwa_decode_workspace_bytes", "gfwa_decode", "gfwa_decode_static")

GFWA_BF16, GFWA_F32 = 0, 1

EXPORTS = ("gfwa_gate_prefix", "gfwa_gate_activation_prefix", "gfwa_gate_activation_backward", "gfwa_forward", "gfwa_backward_workspace_bytes", "gfwa_backward_fast_workspace_bytes", "gfwa_backward",
           "gfwa_forward_gqa", "gfwa_backward_gqa", "gfwa_decode_workspace_bytes", "gfwa_decode", "gfwa_decode_static", "gfwa_gate_scan_workspace_bytes", "gfwa_gate_prefix_stp",
           "gfwa_strerror", "gfwa_version", "gfwa_probe_mfma", "gfwa_probe_copy", "gfwa_profile_enable", "gfwa_profile_read",
           "gfwa_profile_kernel_name")
N_KERNELS = 13


class GfwaError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__(f"libgfwa error {code}: {text}")
        self.code = code


def lib_path() -> str:
    return _LIB_PATH


def load_library() -> ctypes.CDLL:
    """Load libgfwa.so, building it first only if no built library exists."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        from .build import build
        build()
    lib = ctypes.CDLL(_LIB_PATH)
    vp, fp, i, f = ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.gfwa_gate_prefix.argtypes = [fp, fp, i, i, i, vp]
    lib.gfwa_gate_prefix.restype = i
    lib.gfwa_gate_activation_prefix.argtypes = [fp, fp, ctypes.c_float, fp, i, i, i, vp]
    lib.gfwa_gate_activation_prefix.restype = i
    lib.gfwa_gate_activation_backward.argtypes = [fp, fp, ctypes.c_float, fp, fp, fp, i, i, i, vp]
    lib.gfwa_gate_activation_backward.restype = i
    lib.gfwa_forward.argtypes = [i, vp, vp, vp, fp, vp, fp, i, i, i, i, i, f, vp]
    lib.gfwa_forward.restype = i
    lib.gfwa_backward_workspace_bytes.argtypes = [i, i, i, i, i, i]
    lib.gfwa_backward_workspace_bytes.restype = ctypes.c_size_t
    lib.gfwa_backward_fast_workspace_bytes.argtypes = [i, i, i, i, i, i]
    lib.gfwa_backward_fast_workspace_bytes.restype = ctypes.c_size_t
    lib.gfwa_backward.argtypes = [i, vp, vp, vp, vp, vp, fp, fp, vp, vp, vp, fp, vp, ctypes.c_size_t,
                                  i, i, i, i, i, f, vp]
    lib.gfwa_backward.restype = i
    lib.gfwa_forward_gqa.argtypes = [i, vp, vp, vp, fp, vp, fp, i, i, i, i, i, i, f, vp]
    lib.gfwa_forward_gqa.restype = i
    lib.gfwa_backward_gqa.argtypes = [i, vp, vp, vp, vp, vp, fp, fp, vp, vp, vp, fp, vp, ctypes.c_size_t,
                                      i, i, i, i, i, i, f, vp]
    lib.gfwa_backward_gqa.restype = i
    lib.gfwa_decode_workspace_bytes.argtypes = [i, i, i, i, i]
    lib.gfwa_decode_workspace_bytes.restype = ctypes.c_size_t
    lib.gfwa_decode.argtypes = [i, vp, vp, vp, fp, fp, vp, vp, fp, vp, ctypes.c_size_t, i, i, i, i, i, i, f, vp]
    lib.gfwa_decode.restype = i
    lib.gfwa_decode_static.argtypes = [i, vp, vp, vp, fp, fp, vp, vp, fp, i, i, i, i, i, i, f, vp]
    lib.gfwa_decode_static.restype = i
    lib.gfwa_gate_scan_workspace_bytes.argtypes = [i, i, i]
    lib.gfwa_gate_scan_workspace_bytes.restype = ctypes.c_size_t
    lib.gfwa_gate_prefix_stp.argtypes = [fp, fp, f, fp, vp, ctypes.c_size_t, i, i, i, vp]
    lib.gfwa_gate_prefix_stp.restype = i
    lib.gfwa_probe_mfma.argtypes = [fp, i, i, i, ctypes.POINTER(ctypes.c_double), vp]
    lib.gfwa_probe_mfma.restype = i
    lib.gfwa_probe_copy.argtypes = [vp, vp, ctypes.c_size_t, vp]
    lib.gfwa_probe_copy.restype = i
    lib.gfwa_strerror.argtypes = [i]
    lib.gfwa_strerror.restype = ctypes.c_char_p
    lib.gfwa_version.argtypes = []
    lib.gfwa_version.restype = i
    lib.gfwa_profile_enable.argtypes = [i]
    lib.gfwa_profile_enable.restype = i
    lib.gfwa_profile_read.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_int), i]
    lib.gfwa_profile_read.restype = i
    lib.gfwa_profile_kernel_name.argtypes = [i]
    lib.gfwa_profile_kernel_name.restype = ctypes.c_char_p
    _lib = lib
    return lib


def _native():
    """The native module, loaded and bound to the library on the first call."""
    global _call
    if _call is None:
        lib = load_library()
        if not os.path.exists(_CALL_PATH):
            from .build import build_binding
            build_binding()
        spec = importlib.util.spec_from_file_location(__package__ + "._gfwa_call", _CALL_PATH)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        module.bind(_check, tuple(ctypes.cast(getattr(lib, n), ctypes.c_void_p).value for n in _CALLED))
        _call = module
    return _call


def gfwa_strerror(code: int) -> str:
    return load_library().gfwa_strerror(int(code)).decode()


def gfwa_version() -> int:
    return int(load_library().gfwa_version())


def _check(code: int) -> None:
    if code != 0:
        raise GfwaError(code, gfwa_strerror(code))


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _need(t: torch.Tensor, shape, dtype, name: str) -> None:
    if not t.is_cuda:
        raise ValueError(f"{name} must live on the GPU")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    if t.dtype != dtype:
        raise TypeError(f"{name} has dtype {t.dtype}, expected {dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")


def gfwa_gate_prefix(alpha: torch.Tensor, c: Optional[torch.Tensor] = None) -> torch.Tensor:
    """c[b,h,t] = sum_{q<=t} alpha[b,h,q];  alpha, c: [B,H,N] fp32 on the GPU."""
    return (_call or _native()).gate_prefix(alpha, c)


def gfwa_gate_activation_prefix(hpre: torch.Tensor, beta: torch.Tensor, eps: float,
                                c: Optional[torch.Tensor] = None) -> torch.Tensor:
    """c = cumsum_t softplus(beta * hpre) / (beta + eps);  hpre, beta, c: [B,H,N] fp32 on the GPU."""
    return (_call or _native()).gate_activation_prefix(hpre, beta, eps, c)


def gfwa_gate_activation_backward(hpre: torch.Tensor, beta: torch.Tensor, eps: float, dalpha: torch.Tensor,
                                  dh: Optional[torch.Tensor] = None, dbeta: Optional[torch.Tensor] = None):
    """(dh, dbeta) from d(alpha); all [B,H,N] fp32 on the GPU."""
    return (_call or _native()).gate_activation_backward(hpre, beta, eps, dalpha, dh, dbeta)


def gfwa_gate_scan_workspace_bytes(B: int, H: int, N: int) -> int:
    return int(load_library().gfwa_gate_scan_workspace_bytes(B, H, N))


def gfwa_gate_prefix_stp(x: torch.Tensor, beta: Optional[torch.Tensor] = None, eps: float = 0.0,
                         c: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    """The prefix by scan-then-propagate (for few, very long rows): of x itself when beta is None, else of
    softplus(beta * x) / (beta + eps).  x, beta, c: [B,H,N] fp32 on the GPU."""
    return (_call or _native()).gate_prefix_stp(x, beta, eps, c, workspace)


def gfwa_forward(Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, c: torch.Tensor, w: int,
                 scale: float, O: Optional[torch.Tensor] = None,
                 L: Optional[torch.Tensor] = None) -> Tuple[torch.Tensor, torch.Tensor]:
    """O, L of the gated sliding-window attention; Q,K,V: [B,H,N,d], c: [B,H,N] fp32."""
    return (_call or _native()).forward(False, Q, K, V, c, w, scale, O, L)


def gfwa_backward_workspace_bytes(dtype: torch.dtype, B: int, H: int, N: int, d: int, w: int) -> int:
    dt = GFWA_BF16 if dtype == torch.bfloat16 else GFWA_F32
    return int(load_library().gfwa_backward_workspace_bytes(dt, B, H, N, d, int(w)))


def gfwa_backward_fast_workspace_bytes(dtype: torch.dtype, B: int, H: int, N: int, d: int, w: int) -> int:
    dt = GFWA_BF16 if dtype == torch.bfloat16 else GFWA_F32
    return int(load_library().gfwa_backward_fast_workspace_bytes(dt, B, H, N, d, int(w)))


def gfwa_backward(Q, K, V, O, dO, c, L, w: int, scale: float, workspace: Optional[torch.Tensor] = None,
                  dQ=None, dK=None, dV=None, dalpha=None):
    """dQ, dK, dV ([B,H,N,d], dtype of Q) and dalpha ([B,H,N] fp32) from the saved O and L.

    workspace: None allocates the minimum; a tensor of gfwa_backward_fast_workspace_bytes selects the
    faster variant of the library (the same holds for gfwa_backward_gqa)."""
    return (_call or _native()).backward(False, Q, K, V, O, dO, c, L, w, scale, workspace, dQ, dK, dV, dalpha)


def gfwa_forward_gqa(Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, c: torch.Tensor, w: int,
                     scale: float, O: Optional[torch.Tensor] = None,
                     L: Optional[torch.Tensor] = None) -> Tuple[torch.Tensor, torch.Tensor]:
    """gfwa_forward with K, V [B,Hkv,N,d]: query head h reads key/value head h // (H // Hkv)."""
    return (_call or _native()).forward(True, Q, K, V, c, w, scale, O, L)


def gfwa_backward_gqa(Q, K, V, O, dO, c, L, w: int, scale: float, workspace: Optional[torch.Tensor] = None,
                      dQ=None, dK=None, dV=None, dalpha=None):
    """gfwa_backward with K, V, dK, dV [B,Hkv,N,d]; dK, dV sum over the query heads of a group."""
    return (_call or _native()).backward(True, Q, K, V, O, dO, c, L, w, scale, workspace, dQ, dK, dV, dalpha)


def gfwa_decode_workspace_bytes(B: int, H: int, T: int, d: int, w: int) -> int:
    return int(load_library().gfwa_decode_workspace_bytes(B, H, T, d, int(w)))


def gfwa_decode(q: torch.Tensor, Kc: torch.Tensor, Vc: torch.Tensor, c: torch.Tensor, pos: torch.Tensor, w: int,
                scale: float, alpha_t: Optional[torch.Tensor] = None, o: Optional[torch.Tensor] = None,
                L: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None):
    """One decoding step: q [B,H,d] against the caches Kc, Vc [B,Hkv,T,d] at positions pos [B] (int32);
    c [B,H,T] fp32 (entry pos is written when alpha_t [B,H] is given).  Returns o [B,H,d], L [B,H]."""
    return (_call or _native()).decode(q, Kc, Vc, c, pos, w, scale, alpha_t, o, L, workspace)


def gfwa_decode_static(q: torch.Tensor, Kc: torch.Tensor, Vc: torch.Tensor, c: torch.Tensor, pos: torch.Tensor,
                       w: int, scale: float, o: torch.Tensor, L: torch.Tensor,
                       alpha_t: Optional[torch.Tensor] = None):
    """gfwa_decode without a workspace and without any allocation: the caller passes the outputs
    o [B,H,d] and L [B,H]; the partial results live in the library's own scratch."""
    return (_call or _native()).decode_static(q, Kc, Vc, c, pos, w, scale, alpha_t, o, L)


def gfwa_probe_mfma(sink: torch.Tensor, iterations: int, workgroups: int, random_operands: int = 0) -> float:
    """Enqueue the bf16 MFMA loop (0: constant operands, 1: pseudo-random operands, 2: pseudo-random operands
    plus one LDS fragment read and five vector instructions per MFMA); returns the floating-point operations
    of the launch."""
    _need(sink, tuple(sink.shape), torch.float32, "sink")
    flops = ctypes.c_double(0.0)
    _check(load_library().gfwa_probe_mfma(sink.data_ptr(), int(iterations), int(workgroups), int(random_operands),
                                          ctypes.byref(flops),
                                          _stream()))
    return float(flops.value)


def gfwa_probe_copy(src: torch.Tensor, dst: torch.Tensor) -> int:
    """Enqueue a plain copy of src into dst (same size, contiguous); returns the bytes copied."""
    if not (src.is_cuda and dst.is_cuda and src.is_contiguous() and dst.is_contiguous()):
        raise ValueError("src and dst must be contiguous GPU tensors")
    nbytes = src.numel() * src.element_size()
    if nbytes != dst.numel() * dst.element_size():
        raise ValueError("src and dst differ in size")
    _check(load_library().gfwa_probe_copy(src.data_ptr(), dst.data_ptr(), nbytes, _stream()))
    return nbytes


def gfwa_profile_enable(on: bool) -> None:
    """Start (clearing old records) or stop per-kernel HIP-event timing inside the library."""
    _check(load_library().gfwa_profile_enable(1 if on else 0))


def gfwa_profile_read() -> dict:
    """{kernel name: (total ms, launches)} for the launches recorded since profiling was enabled."""
    ms = (ctypes.c_float * N_KERNELS)()
    cnt = (ctypes.c_int * N_KERNELS)()
    _check(load_library().gfwa_profile_read(ms, cnt, N_KERNELS))
    return {gfwa_profile_kernel_name(k): (float(ms[k]), int(cnt[k])) for k in range(N_KERNELS)}


def gfwa_profile_kernel_name(k: int) -> str:
    return load_library().gfwa_profile_kernel_name(int(k)).decode()
