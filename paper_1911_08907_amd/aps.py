"""Thin Python binding of libaps.so (argument marshalling only).

The names match the C ABI declared in include/aps.h.  Arrays are torch tensors
on the GPU (torch provides device memory and the current stream); the format
palette is a list of ``Format``.  Every computation happens in the HIP kernels
of libaps.so; if the library is missing, loading fails loudly.
"""
from __future__ import annotations

import ctypes
import functools
import os
from dataclasses import dataclass
from typing import Iterable, Sequence

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libaps.so")

APS_OK = 0
APS_ERR_NULL = -1
APS_ERR_SIZE = -2
APS_ERR_FORMAT = -3
APS_ERR_ALIGN = -4
APS_ERR_UNSUPPORTED = -5
APS_ERR_DEVICE = -6

APS_INPUT_QUANTIZED = 1
APS_OUTPUT_SCALED = 2
APS_MAX_FORMATS = 8

EXPORTS = ("aps_format_supported", "aps_layer_maxabs", "aps_layer_scales", "aps_quantize",
           "aps_sim_reduce", "aps_sim_reduce_ex", "aps_sim_reduce_codes", "aps_dequantize", "aps_lp_gemm",
           "aps_sync_workspace_bytes", "aps_sync_route", "aps_sync", "aps_sync_noalloc", "aps_strerror")

APS_ACC_SEQUENTIAL = 0
APS_ACC_KAHAN = 1

APS_SYNC_PASS1 = 1
APS_SYNC_PASS2 = 2
APS_SYNC_ONE_PASS = 4
APS_SYNC_TWO_PASS = 8
APS_SYNC_GUESS = 16
APS_SYNC_ROUTE_TWO_PASS = 0
APS_SYNC_ROUTE_ONE_PASS = 1
APS_SYNC_ROUTE_GUESS = 2
APS_SYNC_SCRATCH_BYTES = 96 << 20


class ApsError(RuntimeError):
    def __init__(self, fn: str, status: int):
        super().__init__(f"{fn}: {strerror(status)} ({status})")
        self.status = status


class aps_format(ctypes.Structure):
    _fields_ = [("e", ctypes.c_int32), ("m", ctypes.c_int32), ("bias", ctypes.c_int32)]


class aps_reduce_opts(ctypes.Structure):
    _fields_ = [("group", ctypes.c_int32), ("accumulator", ctypes.c_int32)]


@dataclass(frozen=True)
class Format:
    """Custom float: 1 sign bit, e exponent bits, m mantissa bits, bias
    (default 2^(e-1)-1)."""

    e: int
    m: int
    bias: int | None = None

    @property
    def b(self) -> int:
        return (1 << (self.e - 1)) - 1 if self.bias is None else self.bias

    @property
    def bits(self) -> int:
        return 1 + self.e + self.m

    @property
    def emax(self) -> int:
        return (1 << self.e) - 2 - self.b

    def c(self) -> aps_format:
        return aps_format(self.e, self.m, self.b)

    def __str__(self) -> str:
        return f"1-{self.e}-{self.m}" + ("" if self.bias is None else f"/b{self.bias}")


_lib = None


def lib() -> ctypes.CDLL:
    """Load libaps.so (built in-tree by paper_1911_08907_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: run paper_1911_08907_amd.build.build() first")
        L = ctypes.CDLL(LIB_PATH)
        P, i32, i64, u32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint32
        FP = ctypes.POINTER(aps_format)
        sig = {
            "aps_format_supported": (ctypes.c_int, [aps_format]),
            "aps_layer_maxabs": (ctypes.c_int, [P, i32, i64, i64, P, i32, P, P]),
            "aps_layer_scales": (ctypes.c_int, [P, i32, i32, FP, i32, P, P, P]),
            "aps_quantize": (ctypes.c_int, [P, i32, i64, i64, P, i32, P, FP, i32, P, P, P, P]),
            "aps_sim_reduce": (ctypes.c_int, [P, i32, i64, i64, P, i32, P, FP, i32, P, u32, P, P, P]),
            "aps_sim_reduce_codes": (ctypes.c_int, [P, i32, i64, i64, P, i32, P, FP, i32, P, u32, P, P, P]),
            "aps_sim_reduce_ex": (ctypes.c_int, [P, i32, i64, i64, P, i32, P, FP, i32, P, u32,
                                                 ctypes.POINTER(aps_reduce_opts), P, P, P]),
            "aps_dequantize": (ctypes.c_int, [P, P, i64, P, i32, P, FP, i32, P, P, P]),
            "aps_lp_gemm": (ctypes.c_int, [P, i64, P, i64, P, i64, i32, i32, i32, aps_format, aps_format, i32, P]),
            "aps_sync_workspace_bytes": (ctypes.c_uint64, [i64, i32]),
            "aps_sync_route": (ctypes.c_int, [i32, i64, FP, i32, u32]),
            "aps_sync": (ctypes.c_int, [P, i32, i64, i64, P, i32, FP, i32, P, u32, P, P, P, P, ctypes.c_uint64, P]),
            "aps_sync_noalloc": (ctypes.c_int, [P, i32, i64, i64, P, i32, FP, i32, P, u32, P, P, P, P]),
            "aps_strerror": (ctypes.c_char_p, [ctypes.c_int]),
        }
        for name, (res, args) in sig.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def strerror(status: int) -> str:
    return lib().aps_strerror(int(status)).decode()


def format_supported(f: Format) -> int:
    return lib().aps_format_supported(f.c())


# ------------------------------------------------------------ marshalling

# A call's marshalling is host time that a small set's two launches (8 us)
# cannot hide: addresses go to ctypes as integers, the dtype tuples are made
# once, and the current stream is asked for as a handle (0.1 us) instead of a
# Stream object (2.8 us).  aps_sync of a small set on MI355X: 19 us a call with
# the objects, 12 without.

def _ptr(t):
    if t is None or isinstance(t, int):
        return t
    return t.data_ptr()


def _stream(stream, dev=None):
    """The hipStream_t to launch on: the given stream, or torch's current
    stream.  The library launches on the current device, so the arrays'
    device must be the current one (and a torch stream's device)."""
    import torch
    cur = None
    if dev is not None and dev.type == "cuda":
        cur = torch.cuda.current_device()
        if (dev.index if dev.index is not None else cur) != cur:
            raise ValueError(f"the arrays are on {dev}, the current device is cuda:{cur}")
        if stream is not None and not isinstance(stream, int) and stream.device != torch.device("cuda", cur):
            raise ValueError(f"the stream is on {stream.device}, the arrays on {dev}")
    if stream is None:
        if cur is None:
            cur = torch.cuda.current_device()
        # the accessor that torch's own compiled code uses; not public, so not relied on
        raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        return raw(cur) if raw is not None else torch.cuda.current_stream(cur).cuda_stream
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _palette(fmts) -> tuple:
    fmts = [fmts.c()] if isinstance(fmts, Format) else [f.c() for f in fmts]
    return (aps_format * max(1, len(fmts)))(*fmts), len(fmts)


def _check(fn: str, st: int):
    if st != APS_OK:
        raise ApsError(fn, st)


@functools.lru_cache(maxsize=None)
def _dtypes(*names):
    import torch
    return tuple(getattr(torch, nm) for nm in names if hasattr(torch, nm))


def _dev_of(*ts):
    """The device of the first tensor among ts (raw int addresses and None
    are skipped), or None."""
    for t in ts:
        if t is not None and not isinstance(t, int):
            return t.device
    return None


def _need(t, name: str, dtypes, numel: int = 0, dev=None, optional: bool = False) -> None:
    """The library reads and writes device memory through raw pointers:
    refuse, before anything reaches it, a tensor that is not on the GPU, not
    of one of ``dtypes``, not contiguous, on another device than ``dev`` or
    smaller than ``numel`` elements.  A raw int address is the caller's
    responsibility."""
    if t is None:
        if optional:
            return
        raise ValueError(f"{name} is required")
    if isinstance(t, int):
        return
    if not getattr(t, "is_cuda", False):
        raise ValueError(f"{name} must be a GPU tensor, got one on {t.device}")
    if dev is not None and t.device != dev:
        raise ValueError(f"{name} is on {t.device}, the other arrays on {dev}")
    if t.dtype not in dtypes:
        raise ValueError(f"{name} must be of dtype {' or '.join(str(d) for d in dtypes)}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if t.numel() < numel:
        raise ValueError(f"{name} has {t.numel()} elements, needs at least {numel}")


def _rows(G, n: int | None = None, name: str = "G"):
    """W and the row stride ld of a [W][ld] fp32 GPU tensor with unit column
    stride and at least n columns."""
    if not isinstance(G, int) and (G is None or not getattr(G, "is_cuda", False)):
        raise ValueError(f"{name} must be a GPU tensor" + ("" if G is None else f", got one on {G.device}"))
    if G.dim() != 2:
        raise ValueError(f"{name}: expected a [W][ld] tensor")
    if G.dtype not in _dtypes("float32"):
        raise ValueError(f"{name} must be float32, got {G.dtype}")
    if G.shape[1] > 1 and G.stride(1) != 1:
        raise ValueError(f"{name} needs unit column stride")
    if n is not None and G.shape[1] < n:
        raise ValueError(f"{name} has {G.shape[1]} columns, fewer than n = {n}")
    return G.shape[0], G.stride(0)


def _layers(offsets, dev) -> int:
    _need(offsets, "offsets", _dtypes("int64"), 1, dev)
    return offsets.numel() - 1


def _code_bytes_of(fmts, count: int) -> int:
    """Bytes of count packed codes of the palette's widest format."""
    bits = max(f.bits for f in ([fmts] if isinstance(fmts, Format) else fmts))
    return code_bytes(count, bits)


_F32 = ("float32",)
_I32 = ("int32",)
_U8 = ("uint8",)
_BITS = ("int32", "uint32")


def _reduce_arrays(dev, L: int, n: int, fmts, scale_exp, fmt_idx, out, codes_out) -> None:
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev, optional=True)
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    _need(out, "out", _dtypes(*_F32), n, dev, optional=True)
    _need(codes_out, "codes_out", _dtypes(*_U8), _code_bytes_of(fmts, n), dev, optional=True)


# ------------------------------------------------------------ entry points
# Each takes torch tensors on the current device; ``n`` is the gradient
# length and ``offsets`` an int64 tensor of L+1 layer boundaries.

def aps_layer_maxabs(G, n: int, offsets, maxabs_bits, stream=None) -> None:
    W, ld = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    _need(maxabs_bits, "maxabs_bits", _dtypes(*_BITS), L, dev)
    _check("aps_layer_maxabs", lib().aps_layer_maxabs(_ptr(G), W, ld, n, _ptr(offsets), L,
                                                      _ptr(maxabs_bits), _stream(stream, dev)))


def aps_layer_scales(maxabs_bits, N: int, fmts, fmt_idx, scale_exp, stream=None) -> None:
    dev = _dev_of(maxabs_bits)
    _need(maxabs_bits, "maxabs_bits", _dtypes(*_BITS), 1, dev)
    L = maxabs_bits.numel()
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev)
    pal, nf = _palette(fmts)
    _check("aps_layer_scales", lib().aps_layer_scales(_ptr(maxabs_bits), maxabs_bits.numel(), int(N), pal,
                                                      nf, _ptr(fmt_idx), _ptr(scale_exp), _stream(stream, dev)))


def aps_quantize(X, n: int, offsets, scale_exp, fmts, fmt_idx, Q=None, codes=None, stream=None) -> None:
    W, ld = _rows(X, n, "X")
    dev = X.device
    L = _layers(offsets, dev)
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev, optional=True)
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    if Q is not None and not isinstance(Q, int):
        _rows(Q, n, "Q")
        if Q.device != dev or Q.shape[0] < W or Q.stride(0) != ld:
            raise ValueError("Q must have X's row stride, at least X's rows and X's device")
    _need(codes, "codes", _dtypes(*_U8), W * _code_bytes_of(fmts, ld), dev, optional=True)
    pal, nf = _palette(fmts)
    _check("aps_quantize", lib().aps_quantize(_ptr(X), W, ld, n, _ptr(offsets), L, _ptr(scale_exp), pal, nf,
                                              _ptr(fmt_idx), _ptr(Q), _ptr(codes), _stream(stream, dev)))


def aps_sim_reduce(G, n: int, offsets, scale_exp, fmts, fmt_idx, flags: int = 0, out=None,
                   codes_out=None, stream=None) -> None:
    W, ld = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    _reduce_arrays(dev, L, n, fmts, scale_exp, fmt_idx, out, codes_out)
    pal, nf = _palette(fmts)
    _check("aps_sim_reduce", lib().aps_sim_reduce(_ptr(G), W, ld, n, _ptr(offsets), L, _ptr(scale_exp), pal,
                                                  nf, _ptr(fmt_idx), int(flags), _ptr(out), _ptr(codes_out),
                                                  _stream(stream, dev)))


def aps_sim_reduce_ex(G, n: int, offsets, scale_exp, fmts, fmt_idx, flags: int = 0, group: int | None = None,
                      accumulator: int = APS_ACC_SEQUENTIAL, out=None, codes_out=None, stream=None) -> None:
    """aps_sim_reduce with the hierarchical-all-reduce order (group size k)
    and a plain or Kahan low-precision accumulator."""
    W, ld = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    _reduce_arrays(dev, L, n, fmts, scale_exp, fmt_idx, out, codes_out)
    pal, nf = _palette(fmts)
    opts = aps_reduce_opts(W if group is None else int(group), int(accumulator))
    _check("aps_sim_reduce_ex", lib().aps_sim_reduce_ex(_ptr(G), W, ld, n, _ptr(offsets), L, _ptr(scale_exp), pal,
                                                        nf, _ptr(fmt_idx), int(flags), ctypes.byref(opts),
                                                        _ptr(out), _ptr(codes_out), _stream(stream, dev)))


def aps_sim_reduce_codes(codes, W: int, ld: int, n: int, offsets, scale_exp, fmts, fmt_idx, flags: int = 0,
                         out=None, codes_out=None, stream=None) -> None:
    """codes: a uint8 tensor holding W rows of packed codes (row stride: the
    code bytes of ld elements)."""
    dev = _dev_of(codes)
    _need(codes, "codes", _dtypes(*_U8), int(W) * _code_bytes_of(fmts, int(ld)), dev)
    if int(ld) < n:
        raise ValueError(f"ld = {ld} is below n = {n}")
    L = _layers(offsets, dev)
    _reduce_arrays(dev, L, n, fmts, scale_exp, fmt_idx, out, codes_out)
    pal, nf = _palette(fmts)
    _check("aps_sim_reduce_codes", lib().aps_sim_reduce_codes(_ptr(codes), int(W), int(ld), n, _ptr(offsets), L,
                                                              _ptr(scale_exp), pal, nf, _ptr(fmt_idx), int(flags),
                                                              _ptr(out), _ptr(codes_out), _stream(stream, dev)))


def aps_dequantize(Q, codes, n: int, offsets, scale_exp, fmts, fmt_idx, out, stream=None) -> None:
    dev = _dev_of(Q, codes, out)
    _need(Q, "Q", _dtypes(*_F32), n, dev, optional=True)
    _need(codes, "codes", _dtypes(*_U8), _code_bytes_of(fmts, n), dev, optional=True)
    _need(out, "out", _dtypes(*_F32), n, dev)
    L = _layers(offsets, dev)
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev, optional=True)
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    pal, nf = _palette(fmts)
    _check("aps_dequantize", lib().aps_dequantize(_ptr(Q), _ptr(codes), n, _ptr(offsets), L, _ptr(scale_exp),
                                                  pal, nf, _ptr(fmt_idx), _ptr(out), _stream(stream, dev)))


def aps_lp_gemm(A, B, fin: Format, facc: Format, accumulator: int = APS_ACC_SEQUENTIAL, C=None,
                stream=None):
    """C = A @ B on a low-precision multiply-accumulate unit: A [M][K] and
    B [K][N] row-major fp32 device tensors (row strides from the tensors),
    inputs cast to ``fin``, products and partial sums rounded to ``facc``."""
    import torch

    for name, t in (("A", A), ("B", B), ("C", C)):
        if t is None and name == "C":
            continue
        if not getattr(t, "is_cuda", False):
            raise ValueError(f"{name} must be a GPU tensor")
        if t.dtype != torch.float32 or t.dim() != 2:
            raise ValueError(f"{name} must be a 2-D float32 tensor")
        if t.device != A.device:
            raise ValueError(f"{name} is on {t.device}, A on {A.device}")
    M, K = A.shape
    K2, N = B.shape
    if K != K2:
        raise ValueError(f"inner dimensions differ: {K} vs {K2}")
    if C is not None and tuple(C.shape) != (M, N):
        raise ValueError(f"C has shape {tuple(C.shape)}, the product {(M, N)}")
    def ld(t, rows, cols):  # row stride; an empty or one-row tensor may report anything
        if rows <= 1 or cols == 0:
            return max(cols, 1)
        if cols > 1 and t.stride(1) != 1:
            raise ValueError("A, B and C need unit column stride")
        return t.stride(0)

    if C is None:
        C = torch.empty((M, N), dtype=torch.float32, device=A.device)
    lda, ldb, ldc = ld(A, M, K), ld(B, K, N), ld(C, M, N)
    _check("aps_lp_gemm", lib().aps_lp_gemm(_ptr(A), lda, _ptr(B), ldb, _ptr(C), ldc, M, N, K, fin.c(),
                                            facc.c(), int(accumulator), _stream(stream, A.device)))
    return C


def aps_sync_workspace_bytes(n: int, L: int) -> int:
    return int(lib().aps_sync_workspace_bytes(int(n), int(L)))


def aps_sync_route(W: int, n: int, fmts, flags: int = 0) -> int:
    """The route aps_sync takes for W workers, n elements and this palette
    (only the route bits of ``flags`` matter): one of APS_SYNC_ROUTE_*.  A
    small set of one format, without a route bit and with both passes in one
    call, may run as two launches of its own instead (see aps.h)."""
    pal, nf = _palette(fmts)
    st = lib().aps_sync_route(int(W), int(n), pal, nf, int(flags))
    if st < 0:
        raise ApsError("aps_sync_route", st)
    return st


def aps_sync(G, n: int, offsets, fmts, fmt_idx=None, flags: int = APS_SYNC_PASS1 | APS_SYNC_PASS2,
             maxabs_bits=None, scale_exp=None, out=None, workspace=None, stream=None):
    """One APS synchronisation in one call (N = W): max-abs, scales and the
    rounded W-worker sum, reading G once where the library can.  ``flags``
    selects the passes and optionally the route.  Missing output or
    workspace tensors are allocated here.  Returns
    (out, scale_exp, maxabs_bits, workspace)."""
    import torch
    W, ld = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    if maxabs_bits is None:
        maxabs_bits = torch.empty(L, dtype=torch.int32, device=dev)
    if scale_exp is None:
        scale_exp = torch.empty(L, dtype=torch.int32, device=dev)
    if out is None:
        out = torch.empty(max(n, 1), dtype=torch.float32, device=dev)[:n]
    if workspace is None:
        workspace = torch.empty(aps_sync_workspace_bytes(n, L), dtype=torch.uint8, device=dev)
    _need(maxabs_bits, "maxabs_bits", _dtypes(*_BITS), L, dev)
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev)
    _need(out, "out", _dtypes(*_F32), n, dev)
    _need(workspace, "workspace", _dtypes(*_U8), 0, dev)
    pal, nf = _palette(fmts)
    _check("aps_sync", lib().aps_sync(_ptr(G), W, ld, n, _ptr(offsets), L, pal, nf, _ptr(fmt_idx), int(flags),
                                      _ptr(maxabs_bits), _ptr(scale_exp), _ptr(out), _ptr(workspace),
                                      workspace.numel() * workspace.element_size(), _stream(stream, dev)))
    return out, scale_exp, maxabs_bits, workspace


def aps_sync_noalloc(G, n: int, offsets, fmts, fmt_idx, maxabs_bits, scale_exp, out,
                     flags: int = APS_SYNC_PASS1 | APS_SYNC_PASS2, stream=None) -> None:
    """aps_sync with the library's static per-GPU workspace instead of a
    caller's (nothing is allocated, here or in the library): every output
    tensor is the caller's."""
    W, ld = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    _need(fmt_idx, "fmt_idx", _dtypes(*_U8), L, dev, optional=True)
    _need(maxabs_bits, "maxabs_bits", _dtypes(*_BITS), L, dev)
    _need(scale_exp, "scale_exp", _dtypes(*_I32), L, dev)
    _need(out, "out", _dtypes(*_F32), n, dev)
    pal, nf = _palette(fmts)
    _check("aps_sync_noalloc", lib().aps_sync_noalloc(_ptr(G), W, ld, n, _ptr(offsets), L, pal, nf, _ptr(fmt_idx),
                                                      int(flags), _ptr(maxabs_bits), _ptr(scale_exp), _ptr(out),
                                                      _stream(stream, dev)))


def code_bytes(count: int, bits: int) -> int:
    """Bytes of a packed code array of ``count`` elements."""
    if bits <= 4:
        return (count + 1) // 2
    if bits <= 8:
        return count
    return 2 * count


# ------------------------------------------------------------ convenience

def aps_step(G, n: int, offsets, fmts, fmt_idx=None, N: int | None = None, flags: int = 0, stream=None):
    """One full APS synchronisation of W simulated workers (Algorithm 1):
    max-abs, scales, fused scale/cast/rounded-sum/unscale.  Returns
    (out, scale_exp, maxabs_bits) as new device tensors."""
    import torch
    W, _ = _rows(G, n)
    dev = G.device
    L = _layers(offsets, dev)
    maxabs = torch.empty(L, dtype=torch.int32, device=dev)
    scale = torch.empty(L, dtype=torch.int32, device=dev)
    out = torch.empty(max(n, 1), dtype=torch.float32, device=dev)[:n]
    aps_layer_maxabs(G, n, offsets, maxabs, stream)
    aps_layer_scales(maxabs, W if N is None else N, fmts, fmt_idx, scale, stream)
    aps_sim_reduce(G, n, offsets, scale, fmts, fmt_idx, flags, out, None, stream)
    return out, scale, maxabs
