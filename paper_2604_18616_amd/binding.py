"""ctypes binding of the C-ABI attention library (argument marshalling only).

Function names mirror include/attn.h.  Tensors are torch CUDA tensors (PyTorch is
used for device memory and streams only); their device pointers and the current
stream handle are passed straight to the library.  There is no fallback: if the
HIP library is missing or fails, the call raises.
"""
from __future__ import annotations

import ctypes
import os

from .build import LIB_PATH, NATIVE_PATH, build_library, stale_sources

_lib = None


class AttnError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__("attn_fwd failed (%d): %s" % (code, msg))
        self.code = code


def load_library(build_if_missing: bool = True):
    """Load libattn_mi355x.so (building it first only if no built library exists; a library older than its
    sources is loaded as it is, with a warning: rebuild with `python -m paper_2604_18616_amd.build`)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            if not build_if_missing:
                raise FileNotFoundError(LIB_PATH)
            build_library()
        elif stale_sources():
            import warnings
            warnings.warn("libattn_mi355x.so is older than %s: rebuild it" % ", ".join(stale_sources()))
        lib = ctypes.CDLL(LIB_PATH)
        i, f, p = ctypes.c_int, ctypes.c_float, ctypes.c_void_p
        lib.attn_fwd.restype = i
        lib.attn_fwd.argtypes = [p, p, p, p, p, i, i, i, i, i, i, i, f, p]
        lib.attn_fwd_tile.restype = i
        lib.attn_fwd_tile.argtypes = [p, p, p, p, p, i, i, i, i, i, i, i, f, i, p]
        lib.attn_fwd_strided.restype = i
        lib.attn_fwd_strided.argtypes = [p, p, p, p, p, i, i, i, i, i, i, p, p, p, p, i, f, p]
        lib.attn_fwd_workspace_bytes.restype = ctypes.c_size_t
        lib.attn_fwd_workspace_bytes.argtypes = [i, i, i, i, i, i]
        lib.attn_fwd_workspace.restype = i
        lib.attn_fwd_workspace.argtypes = [p, p, p, p, p, i, i, i, i, i, i, p, p, p, p, i, f, p, ctypes.c_size_t, i, p]
        ll = ctypes.c_longlong
        lib.gemm_bf16.restype = i
        lib.gemm_bf16.argtypes = [p, p, p, i, i, i, ll, ll, ll, i, p]
        lib.gemm_bf16_tile.restype = i
        lib.gemm_bf16_tile.argtypes = [p, p, p, i, i, i, ll, ll, ll, i, i, p]
        lib.gemm_bf16_workspace_bytes.restype = ctypes.c_size_t
        lib.gemm_bf16_workspace_bytes.argtypes = [i, i, i]
        lib.gemm_bf16_workspace.restype = i
        lib.gemm_bf16_workspace.argtypes = [p, p, p, i, i, i, ll, ll, ll, i, i, i, p, ctypes.c_size_t, p]
        lib.gemm_bf16_auto_tile.restype = i
        lib.gemm_bf16_auto_tile.argtypes = [i, i]
        lib.gemm_bf16_flops.restype = ctypes.c_double
        lib.gemm_bf16_flops.argtypes = [i, i, i]
        lib.moe_ffn_fp8_workspace_bytes.restype = ctypes.c_size_t
        lib.moe_ffn_fp8_workspace_bytes.argtypes = [i, i, i, i, i]
        lib.moe_ffn_fp8_workspace_offset.restype = ctypes.c_longlong
        lib.moe_ffn_fp8_workspace_offset.argtypes = [i, i, i, i, i, i]
        lib.moe_ffn_fp8.restype = i
        lib.moe_ffn_fp8.argtypes = [p, p, p, p, p, p, p, p, i, i, i, i, i, p, ctypes.c_size_t, p]
        lib.moe_ffn_fp8_ex.restype = i
        lib.moe_ffn_fp8_ex.argtypes = [p, p, p, p, p, p, p, p, i, i, i, i, i, p, ctypes.c_size_t, i, i, i, p]
        lib.moe_ffn_fp8_static.restype = i
        lib.moe_ffn_fp8_static.argtypes = [p, p, p, p, p, p, p, p, i, i, i, i, i, p]
        lib.moe_ffn_fp8_flops_per_pair.restype = ctypes.c_double
        lib.moe_ffn_fp8_flops_per_pair.argtypes = [i, i]
        lib.attn_strerror.restype = ctypes.c_char_p
        lib.attn_strerror.argtypes = [i]
        lib.attn_version.restype = i
        lib.attn_version.argtypes = []
        lib.attn_fwd_flops.restype = ctypes.c_double
        lib.attn_fwd_flops.argtypes = [i, i, i, i, i, i, i]
        lib.attn_mfma_calibration.restype = ctypes.c_double
        lib.attn_mfma_calibration.argtypes = [p, i, i, p]
        lib.attn_mfma_calibration_data.restype = ctypes.c_double
        lib.attn_mfma_calibration_data.argtypes = [p, i, i, i, p]
        lib.attn_device_info.restype = i
        lib.attn_device_info.argtypes = [i, ctypes.POINTER(i), ctypes.POINTER(i), ctypes.POINTER(ctypes.c_double)]
        _lib = lib
    return _lib


_native = None


def _load_native():
    """The extension module that makes the plain calls (csrc/native_calls.cpp), with the library's addresses; False, with a
    warning, where it has not been built or not for this torch: the calls then take the longer way through this file, to the
    same kernels."""
    global _native
    import importlib.util
    import warnings

    import torch
    lib = load_library()
    try:
        if not os.path.exists(NATIVE_PATH):
            raise ImportError("it has not been built")
        spec = importlib.util.spec_from_file_location(__package__ + "._native", NATIVE_PATH)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        if module.torch_version != torch.__version__:
            raise ImportError("it was built for torch %s" % module.torch_version)
    except ImportError as why:
        warnings.warn("calls take longer without the extension module (python -m paper_2604_18616_amd.build builds it): %s" % why)
        module = False
    if module:
        module.bind(*(ctypes.cast(f, ctypes.c_void_p).value for f in (
            lib.attn_fwd, lib.attn_fwd_strided, lib.attn_fwd_workspace_bytes, lib.attn_fwd_workspace,
            lib.gemm_bf16_workspace_bytes, lib.gemm_bf16_tile, lib.gemm_bf16_workspace)))
    _native = module
    return module


def strerror(code: int) -> str:
    return load_library().attn_strerror(int(code)).decode()


def version() -> int:
    return load_library().attn_version()


def device_info(device: int = 0) -> dict:
    """Compute units, maximum shader clock and the bf16 matrix peak that follows (attn_device_info)."""
    cus, khz, peak = ctypes.c_int(0), ctypes.c_int(0), ctypes.c_double(0.0)
    rc = load_library().attn_device_info(int(device), ctypes.byref(cus), ctypes.byref(khz), ctypes.byref(peak))
    if rc != 0:
        raise AttnError(rc, strerror(rc))
    return {"cus": cus.value, "clock_mhz": khz.value / 1e3, "bf16_peak_tflops_from_props": peak.value}


def attn_fwd_flops(B, Hq, Hkv, Sq, Sk, D, causal) -> float:
    return load_library().attn_fwd_flops(B, Hq, Hkv, Sq, Sk, D, int(bool(causal)))


def attn_fwd_raw(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, Hq, Hkv, Sq, Sk, D, causal, scale, stream_ptr, wg_rows=0) -> int:
    """Direct call with integer device addresses; returns the library's status code.  wg_rows != 0 goes
    through attn_fwd_tile (workgroup shape forced: 128 or 256 query rows)."""
    lib = load_library()
    if wg_rows:
        return lib.attn_fwd_tile(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, Hq, Hkv, Sq, Sk, D,
                                 int(bool(causal)), float(scale), int(wg_rows), stream_ptr)
    return lib.attn_fwd(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, Hq, Hkv, Sq, Sk, D,
                        int(bool(causal)), float(scale), stream_ptr)


_Int64x3 = ctypes.c_longlong * 3


def _strides3(t):
    return _Int64x3(*t.stride()[:3])


def _streams(t, stream):
    """(handle to launch on, whether torch's memory for t's device may be used on it without keeping it alive).  Handles
    instead of Stream objects: making one is a large part of the host time of a small call."""
    import torch
    current = torch._C._cuda_getCurrentRawStream(t.get_device())
    if stream is None:
        return current, True
    handle = stream.cuda_stream
    return handle, handle == current


def _scratch(need, device):
    """Torch memory for a call's parts; None where there is none left: such a call runs uncut, as it would without it."""
    import torch
    try:
        return torch.empty(need, dtype=torch.uint8, device=device)
    except torch.cuda.OutOfMemoryError:
        return None


_torch_scratch = _scratch


def _plain_calls(t):
    """The extension module for a call whose first tensor is t; False without it, and where a program has put its own source
    of memory for the parts in place of _scratch, which only the code below asks.  Tensors on the CPU are refused without loading anything."""
    if _scratch is not _torch_scratch:
        return False
    if _native is None:
        return _load_native() if getattr(t, "is_cuda", False) else False
    return _native


def attn_fwd(q, k, v, o=None, lse=None, causal=False, scale=None, stream=None):
    """O, LSE = attention forward of bf16 CUDA tensors q [B,Hq,Sq,D], k/v [B,Hkv,Sk,D].

    The tensors may be strided views (e.g. a [B,S,H,D] buffer transposed to [B,H,S,D]) as long
    as the last dimension is contiguous; contiguous inputs take attn_fwd, anything else
    attn_fwd_strided.  o (bf16, q's shape) and lse (fp32 [B,Hq,Sq], contiguous) are allocated
    with torch if not given.  The kernel is enqueued on `stream` (default: torch's current
    stream); no sync.
    """
    if o is None and lse is None and stream is None:
        native = _plain_calls(q)
        done = native.attn(q, k, v, causal, scale) if native else None         # None: not a plain call
        if done is not None:
            if type(done) is int:
                raise AttnError(done, strerror(done))
            return done
    import torch

    if not (q.is_cuda and k.is_cuda and v.is_cuda):
        raise ValueError("q, k, v must be CUDA tensors: there is no CPU path")
    bf16 = torch.bfloat16
    qst, kst, vst = q.stride(), k.stride(), v.stride()
    if (q.dtype != bf16 or k.dtype != bf16 or v.dtype != bf16 or len(qst) != 4 or len(kst) != 4 or len(vst) != 4
            or qst[3] != 1 or kst[3] != 1 or vst[3] != 1):
        raise ValueError("q, k, v must be 4-D bfloat16 tensors with a contiguous last dimension")
    qs, ks = q.shape, k.shape
    B, Hq, Sq, D = qs
    Bk, Hkv, Sk, Dk = ks
    if v.shape != ks or Bk != B or Dk != D:
        raise ValueError("inconsistent q/k/v shapes")
    device = q.device
    if o is None:
        o = torch.empty_like(q)          # keeps q's layout for dense views
    elif o.shape != qs or o.dtype != bf16:
        raise ValueError("o must be bfloat16 with q's shape and a contiguous last dimension")
    ost = o.stride()
    if ost[3] != 1:
        raise ValueError("o must be bfloat16 with q's shape and a contiguous last dimension")
    if lse is None:
        lse = torch.empty((B, Hq, Sq), dtype=torch.float32, device=device)
    elif not lse.is_cuda or lse.dtype != torch.float32 or tuple(lse.shape) != (B, Hq, Sq) or not lse.is_contiguous():
        raise ValueError("lse must be a contiguous float32 CUDA tensor of shape [B, Hq, Sq]")
    if k.device != device or v.device != device or o.device != device or lse.device != device:
        raise ValueError("q, k, v, o, lse must live on one CUDA device")
    scale = float(D) ** -0.5 if scale is None else float(scale)
    causal = 1 if causal else 0
    stream, own = _streams(q, stream)
    lib = load_library()
    # few query rows or few heads: cut the keys over workgroups too, with torch's memory for the parts (only on the stream torch
    # will reuse that memory on, and where the byte offsets inside a head fit the 32 bits that the cut works in; elsewhere the
    # call does without it)
    need = lib.attn_fwd_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) if own and (Sq <= 64 or B * Hq * Sq <= 160 * 128) else 0
    ws = _scratch(need, device) if need and (Sk + 64) * (kst[2] if kst[2] > vst[2] else vst[2]) < 1 << 31 else None
    if ws is not None:
        rc = lib.attn_fwd_workspace(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(),
                                    B, Hq, Hkv, Sq, Sk, D, _Int64x3(*qst[:3]), _Int64x3(*kst[:3]), _Int64x3(*vst[:3]), _Int64x3(*ost[:3]),
                                    causal, scale, ws.data_ptr(), need, need // (4 * B * Hq * Sq * (D + 2)), stream)
    elif q.is_contiguous() and k.is_contiguous() and v.is_contiguous() and o.is_contiguous():
        rc = lib.attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(),
                          B, Hq, Hkv, Sq, Sk, D, causal, scale, stream)
    else:
        rc = lib.attn_fwd_strided(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(),
                                  B, Hq, Hkv, Sq, Sk, D, _Int64x3(*qst[:3]), _Int64x3(*kst[:3]), _Int64x3(*vst[:3]), _Int64x3(*ost[:3]),
                                  causal, scale, stream)
    if rc != 0:
        raise AttnError(rc, strerror(rc))
    return o, lse


def _aligned(a, b, c):
    """Whether the rows of three matrices start at multiples of 16 bytes."""
    return not ((a.data_ptr() | b.data_ptr() | c.data_ptr()) & 15 or (a.stride(0) | b.stride(0) | c.stride(0)) & 7)


def gemm_bf16(a, b, c=None, b_is_nk=False, stream=None, tile=0):
    """C = A B for bf16 CUDA tensors a [M,K] and b [K,N] (or [N,K] if b_is_nk); rows contiguous,
    row pitch free.  c (bf16 [M,N]) is allocated with torch if not given.  Enqueued on `stream`
    (default: torch's current stream); no sync.  tile: 0 (by size) or a shape code of gemm.h: 64, 128, 1284, 256, 2564, those with 16 appended, or 19216 (gemm_bf16_tile)."""
    if c is None and stream is None and tile == 0:
        native = _plain_calls(a)
        done = native.gemm(a, b, b_is_nk) if native else None
        if done is not None:
            if type(done) is int:
                raise AttnError(done, strerror(done))
            return done
    import torch

    if not (a.is_cuda and b.is_cuda):
        raise ValueError("a, b must be CUDA tensors: there is no CPU path")
    for t in (a, b):
        if t.dtype != torch.bfloat16 or t.dim() != 2 or t.stride(1) != 1:
            raise ValueError("a, b must be 2-D bfloat16 tensors with contiguous rows")
    M, K = a.shape
    N = b.shape[0] if b_is_nk else b.shape[1]
    if (b.shape[1] if b_is_nk else b.shape[0]) != K:
        raise ValueError("inner dimensions differ")
    if c is None:
        c = torch.empty((M, N), dtype=torch.bfloat16, device=a.device)
    elif c.shape != (M, N) or c.dtype != torch.bfloat16 or c.stride(1) != 1:
        raise ValueError("c must be bfloat16 [M,N] with contiguous rows")
    stream, own = _streams(a, stream)
    lib = load_library()
    # results of few tiles: cut k over workgroups too, with torch's memory for the parts (only on the stream torch will
    # reuse that memory on, and for operands of the aligned kernel; elsewhere the call does without it)
    need = lib.gemm_bf16_workspace_bytes(M, N, K) if tile == 0 and own else 0
    ws = _scratch(need, a.device) if need and _aligned(a, b, c) else None
    if ws is not None:
        rc = lib.gemm_bf16_workspace(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, a.stride(0), b.stride(0), c.stride(0),
                                     1 if b_is_nk else 0, 0, 0, ws.data_ptr(), need, stream)
    else:
        rc = lib.gemm_bf16_tile(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, a.stride(0), b.stride(0), c.stride(0),
                                1 if b_is_nk else 0, int(tile), stream)
    if rc != 0:
        raise AttnError(rc, strerror(rc))
    return c


def moe_workspace_bytes(T, H, I, E, KTOP) -> int:
    return int(load_library().moe_ffn_fp8_workspace_bytes(T, H, I, E, KTOP))


def moe_workspace_offset(T, H, I, E, KTOP, part: int) -> int:
    return int(load_library().moe_ffn_fp8_workspace_offset(T, H, I, E, KTOP, part))


def moe_ffn_fp8(x, ids, wts, w13, s13, w2, s2, y=None, workspace=None, stream=None, row_tile=0):
    """Block-quantized FP8 MoE feed-forward of CUDA tensors: x bf16 [T,H]; ids int32 [T,KTOP] (local
    expert or negative); wts fp32 [T,KTOP]; w13 uint8 [E,2I,H] and w2 uint8 [E,H,I] (e4m3 codes);
    s13 fp32 [E,2I/128,H/128]; s2 fp32 [E,H/128,I/128].  y (bf16 [T,H]) and the workspace (uint8, at
    least moe_workspace_bytes(...)) are allocated with torch if not given.  Enqueued on `stream`
    (default: torch's current stream); no sync.  row_tile: 0 (by the rows the experts get), 128 or 64 (moe_ffn_fp8_ex)."""
    import torch

    for t in (x, ids, wts, w13, s13, w2, s2):
        if not t.is_cuda or not t.is_contiguous():
            raise ValueError("all MoE tensors must be contiguous CUDA tensors: there is no CPU path")
    T, H = x.shape
    E, I2, _ = w13.shape
    I, K = I2 // 2, ids.shape[1]
    if (x.dtype != torch.bfloat16 or ids.dtype != torch.int32 or wts.dtype != torch.float32 or w13.dtype != torch.uint8
            or w2.dtype != torch.uint8 or s13.dtype != torch.float32 or s2.dtype != torch.float32):
        raise ValueError("dtypes: x bf16, ids int32, wts/s13/s2 fp32, w13/w2 uint8")
    if (w13.shape != (E, 2 * I, H) or w2.shape != (E, H, I) or ids.shape != (T, K) or wts.shape != (T, K)
            or s13.shape != (E, 2 * I // 128, H // 128) or s2.shape != (E, H // 128, I // 128)):
        raise ValueError("inconsistent MoE shapes")
    lib = load_library()
    need = lib.moe_ffn_fp8_workspace_bytes(T, H, I, E, K)
    if y is None:
        y = torch.empty((T, H), dtype=torch.bfloat16, device=x.device)
    if not y.is_cuda or y.dtype != torch.bfloat16 or tuple(y.shape) != (T, H) or not y.is_contiguous():
        raise ValueError("y must be a contiguous bfloat16 CUDA tensor of shape [T, H]")
    stream, own = _streams(x, stream)
    if workspace is None:
        # a temporary is only safe on the stream torch will reuse its memory on: the kernels are still queued
        # when this function returns
        if not own:
            raise ValueError("pass a workspace when `stream` is not torch's current stream")
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=x.device)
    if (not workspace.is_cuda or workspace.dtype != torch.uint8 or not workspace.is_contiguous()
            or workspace.numel() < need or workspace.data_ptr() % 256):
        raise ValueError("workspace must be a contiguous uint8 CUDA tensor of at least moe_workspace_bytes(...) bytes, 256-byte aligned")
    rc = lib.moe_ffn_fp8_ex(x.data_ptr(), ids.data_ptr(), wts.data_ptr(), w13.data_ptr(), s13.data_ptr(), w2.data_ptr(),
                            s2.data_ptr(), y.data_ptr(), T, H, I, E, K, workspace.data_ptr(), workspace.numel(),
                            0, 4, int(row_tile), stream)
    if rc != 0:
        raise AttnError(rc, strerror(rc))
    return y
