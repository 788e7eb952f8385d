"""Binding of libbq.so: the same entry points as include/bq.h, taking torch tensors.  The calls of the path go through the
module bqcall (csrc/bqcall.c) where it is built for this Python, else, as the others do, through ctypes.

Argument marshalling only — every step of the path runs in the library's HIP kernels.  torch is used
for device memory and the current stream, nothing else.  There is no CPU or eager fallback: if the
library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os
from typing import Optional

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libbq.so")
CALL_PATH = os.path.join(HERE, "bqcall" + importlib.machinery.EXTENSION_SUFFIXES[0])  # (the suffix names the Python it is built for)

BQ_OK = 0
BQ_F32, BQ_F16, BQ_BF16 = 0, 1, 2
STATUS_NAMES = {0: "BQ_OK", 1: "BQ_ERR_NULL", 2: "BQ_ERR_SHAPE", 3: "BQ_ERR_DTYPE", 4: "BQ_ERR_ALIGN",
                5: "BQ_ERR_WORKSPACE", 6: "BQ_ERR_UNSUPPORTED", 7: "BQ_ERR_HIP"}
DTYPE_CODES = {"f32": BQ_F32, "f16": BQ_F16, "bf16": BQ_BF16}
RESIDUAL_STEP = {"f16": 2.0 ** -12, "bf16": 1.0}  # bq_residual_split: weight of a piece over the weight of the one before it

EXPORTS = ["bq_plan_bytes", "bq_plan_build", "bq_butterfly_fwd", "bq_butterfly_inv", "bq_butterfly_fwd_quant",
           "bq_butterfly_fwd_fakequant", "bq_hadamard_fwd", "bq_cayley_build", "bq_kron_fwd", "bq_kron_inv",
           "bq_butterfly_bwd_workspace_bytes", "bq_butterfly_bwd", "bq_butterfly_bwd_static",
           "bq_butterfly_bwd_static_max_bytes", "bq_residual_scratch_bytes", "bq_residual_split", "bq_quantiser_grad",
           "bq_probe_copy", "bq_probe_read", "bq_probe_read_sink_bytes",
           "bq_probe_fma", "bq_probe_fma_out_floats",
           "bq_status_string", "bq_last_error",
           "bq_version"]


class bq_rows(ctypes.Structure):
    _fields_ = [("rows", ctypes.c_int64), ("n", ctypes.c_int32), ("heads", ctypes.c_int32),
                ("ld_x", ctypes.c_int64), ("ld_y", ctypes.c_int64), ("dtype", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


class bq_quant(ctypes.Structure):
    _fields_ = [("bits", ctypes.c_int32), ("group", ctypes.c_int32), ("scale_dtype", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


class BqError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"{STATUS_NAMES.get(status, status)}: {text}")
        self.status = status


_LIB = None


def lib() -> ctypes.CDLL:
    """Load libbq.so (built in-tree by paper_2509_09679_amd.build); fails loudly if it is absent."""
    global _LIB
    if _LIB is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(f"{LIB_PATH} not built: run `python -m paper_2509_09679_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        vp, sz = ctypes.c_void_p, ctypes.c_size_t
        L.bq_plan_bytes.argtypes = [ctypes.c_int32, ctypes.c_int32]
        L.bq_plan_bytes.restype = sz
        L.bq_plan_build.argtypes = [vp, ctypes.c_int32, ctypes.c_int32, vp, sz, vp]
        L.bq_plan_build.restype = ctypes.c_int
        for name in ("bq_butterfly_fwd", "bq_butterfly_inv"):
            f = getattr(L, name)
            f.argtypes = [vp, vp, vp, ctypes.POINTER(bq_rows), vp]
            f.restype = ctypes.c_int
        L.bq_hadamard_fwd.argtypes = [vp, vp, ctypes.POINTER(bq_rows), vp]
        L.bq_hadamard_fwd.restype = ctypes.c_int
        L.bq_butterfly_fwd_quant.argtypes = [vp, vp, vp, vp, ctypes.POINTER(bq_quant), ctypes.POINTER(bq_rows), vp]
        L.bq_butterfly_fwd_fakequant.argtypes = [vp, vp, vp, vp, ctypes.POINTER(bq_quant), ctypes.POINTER(bq_rows), vp]
        L.bq_butterfly_fwd_fakequant.restype = ctypes.c_int
        L.bq_cayley_build.argtypes = [vp, ctypes.c_int32, vp, vp]
        L.bq_cayley_build.restype = ctypes.c_int
        for f in (L.bq_kron_fwd, L.bq_kron_inv):
            f.argtypes = [vp, vp, vp, ctypes.c_int32, vp, ctypes.POINTER(bq_rows), vp]
            f.restype = ctypes.c_int
        L.bq_butterfly_fwd_quant.restype = ctypes.c_int
        L.bq_residual_scratch_bytes.argtypes = []
        L.bq_residual_scratch_bytes.restype = sz
        L.bq_residual_split.argtypes = [vp, ctypes.c_int64, ctypes.c_int32, vp, ctypes.c_int32, ctypes.c_int32, vp, vp, vp]
        L.bq_residual_split.restype = ctypes.c_int
        L.bq_quantiser_grad.argtypes = [vp, vp, vp, vp, ctypes.POINTER(bq_quant), ctypes.POINTER(bq_rows), vp]
        L.bq_quantiser_grad.restype = ctypes.c_int
        L.bq_butterfly_bwd_workspace_bytes.argtypes = [ctypes.POINTER(bq_rows)]
        L.bq_butterfly_bwd_workspace_bytes.restype = sz
        L.bq_butterfly_bwd.argtypes = [vp, vp, vp, vp, vp, vp, sz, ctypes.POINTER(bq_rows), vp]
        L.bq_butterfly_bwd.restype = ctypes.c_int
        L.bq_butterfly_bwd_static.argtypes = [vp, vp, vp, vp, vp, ctypes.POINTER(bq_rows), vp]
        L.bq_butterfly_bwd_static.restype = ctypes.c_int
        L.bq_butterfly_bwd_static_max_bytes.argtypes = []
        L.bq_butterfly_bwd_static_max_bytes.restype = sz
        L.bq_probe_copy.argtypes = [vp, vp, sz, vp]
        L.bq_probe_copy.restype = ctypes.c_int
        L.bq_probe_read.argtypes = [vp, sz, vp, vp]
        L.bq_probe_read.restype = ctypes.c_int
        L.bq_probe_read_sink_bytes.argtypes = []
        L.bq_probe_read_sink_bytes.restype = sz
        L.bq_probe_fma.argtypes = [vp, ctypes.c_int32, vp]
        L.bq_probe_fma.restype = ctypes.c_int64
        L.bq_probe_fma_out_floats.argtypes = []
        L.bq_probe_fma_out_floats.restype = sz
        L.bq_status_string.argtypes = [ctypes.c_int]
        L.bq_status_string.restype = ctypes.c_char_p
        L.bq_last_error.restype = ctypes.c_char_p
        L.bq_version.restype = ctypes.c_int
        _LIB = L
    return _LIB


_CALLS = None

# the entry points a program calls per batch, and what their arguments are (csrc/bqcall.c)
_KINDS = {"bq_plan_build": "piipus", "bq_butterfly_fwd": "ppprs", "bq_butterfly_inv": "ppprs", "bq_butterfly_fwd_quant": "ppppqrs",
          "bq_butterfly_fwd_fakequant": "ppppqrs", "bq_kron_fwd": "pppiprs", "bq_kron_inv": "pppiprs", "bq_butterfly_bwd": "ppppppurs"}


def _general_call(name: str, kinds: str):
    """An entry point through its ctypes prototype, with the arguments a Caller takes."""
    fn = getattr(lib(), name)

    def call(*args):
        try:
            return fn(*[_ptr(a) if k == "p" else ctypes.byref(a) if k in "rq" else a for k, a in zip(kinds, args)])
        except ctypes.ArgumentError as e:
            raise TypeError(str(e)) from None

    return call


class _Calls:
    """One callable per entry point of _KINDS, without the "bq_" in front: a Caller, or its ctypes prototype where `path` does not exist."""

    def __init__(self, path: str = CALL_PATH):
        L = lib()
        module = None
        if os.path.exists(path):
            loader = importlib.machinery.ExtensionFileLoader("bqcall", path)
            module = importlib.util.module_from_spec(importlib.util.spec_from_loader("bqcall", loader))
            loader.exec_module(module)
        for name, kinds in _KINDS.items():
            call = _general_call(name, kinds)
            if module:
                call = module.Caller(ctypes.cast(getattr(L, name), ctypes.c_void_p).value, kinds, bq_rows, bq_quant, call)
            setattr(self, name[3:], call)


def _calls() -> _Calls:
    global _CALLS
    if _CALLS is None:
        _CALLS = _Calls()
    return _CALLS


def _check(status: int):
    if status != BQ_OK:
        raise BqError(status, lib().bq_last_error().decode())


def _dtype_code(t) -> int:
    import torch

    return {torch.float32: BQ_F32, torch.float16: BQ_F16, torch.bfloat16: BQ_BF16}[t.dtype]


_current_raw_stream = None


def _stream_ptr(stream=None) -> int:
    """The stream's handle; the current stream's of the current device by default.  torch.cuda.current_stream() builds a Stream
    object for it, 2.8 us of the 7.7 us of host time of a call; asked for the bare handle torch takes 0.15 us."""
    global _current_raw_stream
    if stream is not None:
        return int(stream.cuda_stream)
    if _current_raw_stream is None:
        import torch

        torch.cuda.init()
        device, raw = getattr(torch._C, "_cuda_getDevice", None), getattr(torch._C, "_cuda_getCurrentRawStream", None)
        if device is None or raw is None:  # (not part of torch's public interface)
            _current_raw_stream = lambda: int(torch.cuda.current_stream().cuda_stream)  # noqa: E731
        else:
            _current_raw_stream = lambda: raw(device())  # noqa: E731
    return _current_raw_stream()


def _require(ok: bool, status: int, text: str) -> None:
    if not ok:
        raise BqError(status, text)


def _require_dense(who: str, name: str, t, code: int, count: int) -> None:
    """What the library cannot see in a bare pointer: element type, extent, contiguity."""
    import torch

    if t is None:  # the library's own check
        return
    known = t.dtype in (torch.float32, torch.float16, torch.bfloat16) and _dtype_code(t) == code
    _require(known, 3, f"{who}: {name} is {t.dtype}")
    _require(t.is_contiguous() and t.numel() >= count, 2, f"{who}: {name} must be contiguous with at least {count} elements")


def _ptr(t) -> Optional[int]:
    return None if t is None else int(t.data_ptr())


def make_rows(x, n: int, heads: int, out=None) -> bq_rows:
    """Descriptor for 2-D row tensors (last dimension contiguous)."""
    assert x.dim() == 2 and (x.shape[0] == 0 or x.stride(1) == 1)
    r = bq_rows()
    r.rows, r.n, r.heads = x.shape[0], n, heads
    r.ld_x = x.stride(0) if x.shape[0] > 1 else n * heads
    o = x if out is None else out
    r.ld_y = o.stride(0) if o.shape[0] > 1 else n * heads
    r.dtype = _dtype_code(x)
    return r


def make_kron_rows(x, d2: int) -> bq_rows:
    """Descriptor for bq_kron_fwd / bq_kron_inv: dense rows of d1 * d2 elements, butterfly size d2."""
    assert x.dim() == 2 and x.is_contiguous() and x.shape[1] % d2 == 0
    r = bq_rows()
    r.rows, r.n, r.heads = x.shape[0], d2, 1
    r.ld_x = r.ld_y = x.shape[1]
    r.dtype = _dtype_code(x)
    return r


# --- entry points, same names as the C ABI -----------------------------------------------------

def bq_plan_bytes(n: int, heads: int = 1) -> int:
    return int(lib().bq_plan_bytes(n, heads))


def bq_plan_build(theta, n: int, heads: int, plan, stream=None) -> None:
    """theta: float32 device tensor [heads, log2 n, n/2]; plan: uint8 device tensor of bq_plan_bytes."""
    _check((_CALLS or _calls()).plan_build(theta, n, heads, plan, plan.numel() * plan.element_size(), _stream_ptr(stream)))


def bq_butterfly_fwd(x, y, plan, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).butterfly_fwd(x, y, plan, rows, _stream_ptr(stream)))


def bq_butterfly_inv(y, x, plan, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).butterfly_inv(y, x, plan, rows, _stream_ptr(stream)))


def bq_hadamard_fwd(x, y, rows: bq_rows, stream=None) -> None:
    _check(lib().bq_hadamard_fwd(_ptr(x), _ptr(y), ctypes.byref(rows), _stream_ptr(stream)))


def bq_butterfly_fwd_quant(x, plan, codes, scales, quant: bq_quant, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).butterfly_fwd_quant(x, plan, codes, scales, quant, rows, _stream_ptr(stream)))


def bq_butterfly_fwd_fakequant(x, plan, yq, hist, quant: bq_quant, rows: bq_rows, stream=None) -> None:
    """yq (rows' dtype, or None) and hist (uint64/int64 tensor of 2^bits counters, or None)."""
    _check((_CALLS or _calls()).butterfly_fwd_fakequant(x, plan, yq, hist, quant, rows, _stream_ptr(stream)))


def bq_cayley_build(params, d1: int, q1, stream=None) -> None:
    _check(lib().bq_cayley_build(_ptr(params), d1, _ptr(q1), _stream_ptr(stream)))


def bq_kron_fwd(x, y, q1, d1: int, plan, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).kron_fwd(x, y, q1, d1, plan, rows, _stream_ptr(stream)))


def bq_kron_inv(y, x, q1, d1: int, plan, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).kron_inv(y, x, q1, d1, plan, rows, _stream_ptr(stream)))


def bq_residual_scratch_bytes() -> int:
    return int(lib().bq_residual_scratch_bytes())


def bq_residual_split(e, pieces, result, scratch, stream=None) -> None:
    """e: dense float32 [rows, cols]; pieces: [2 (float16) or 3 (bfloat16), rows, ld], piece p with weight
    RESIDUAL_STEP ** p; result: float32 [2]; scratch: uint8."""
    rows, cols = e.shape
    assert e.is_contiguous() and pieces.is_contiguous() and pieces.shape[0] == (2 if _dtype_code(pieces) == BQ_F16 else 3)
    assert pieces.shape[1] == rows and scratch.numel() * scratch.element_size() >= bq_residual_scratch_bytes()
    _require_dense("bq_residual_split", "e", e, BQ_F32, 0)
    _require_dense("bq_residual_split", "result", result, BQ_F32, 2)
    _check(lib().bq_residual_split(_ptr(e), rows, cols, _ptr(pieces), pieces.shape[2], _dtype_code(pieces), _ptr(result),
                                   _ptr(scratch), _stream_ptr(stream)))


def bq_quantiser_grad(v, vq, g, factor, quant: bq_quant, rows: bq_rows, stream=None) -> None:
    """In place on g (float32); factor: float32 device tensor of one element."""
    count = rows.rows * rows.n * rows.heads
    for name, t, code, least in (("v", v, rows.dtype, count), ("vq", vq, rows.dtype, count), ("g", g, BQ_F32, count),
                                 ("factor", factor, BQ_F32, 1)):
        _require_dense("bq_quantiser_grad", name, t, code, least)
    _check(lib().bq_quantiser_grad(_ptr(v), _ptr(vq), _ptr(g), _ptr(factor), ctypes.byref(quant), ctypes.byref(rows),
                                   _stream_ptr(stream)))


def bq_butterfly_bwd_workspace_bytes(rows: bq_rows) -> int:
    return int(lib().bq_butterfly_bwd_workspace_bytes(ctypes.byref(rows)))


def bq_butterfly_bwd(x, dy, plan, dx, dtheta, workspace, rows: bq_rows, stream=None) -> None:
    _check((_CALLS or _calls()).butterfly_bwd(x, dy, plan, dx, dtheta, workspace, workspace.numel() * workspace.element_size(), rows,
                                              _stream_ptr(stream)))


def bq_butterfly_bwd_static(x, dy, plan, dx, dtheta, rows: bq_rows, stream=None) -> None:
    _check(lib().bq_butterfly_bwd_static(_ptr(x), _ptr(dy), _ptr(plan), _ptr(dx), _ptr(dtheta), ctypes.byref(rows),
                                         _stream_ptr(stream)))


def bq_butterfly_bwd_static_max_bytes() -> int:
    return int(lib().bq_butterfly_bwd_static_max_bytes())


def bq_probe_copy(src, dst, nbytes: int, stream=None) -> None:
    _check(lib().bq_probe_copy(_ptr(src), _ptr(dst), nbytes, _stream_ptr(stream)))


def bq_probe_read_sink_bytes() -> int:
    return int(lib().bq_probe_read_sink_bytes())


def bq_probe_read(src, nbytes: int, sink, stream=None) -> None:
    _check(lib().bq_probe_read(_ptr(src), nbytes, _ptr(sink), _stream_ptr(stream)))


def bq_probe_fma_out_floats() -> int:
    return int(lib().bq_probe_fma_out_floats())


def bq_probe_fma(out, iters: int, stream=None) -> int:
    """Launches the FMA loop; returns the number of lane-FMAs of the launch."""
    n = int(lib().bq_probe_fma(_ptr(out), iters, _stream_ptr(stream)))
    if n < 0:
        raise BqError(7, "bq_probe_fma failed")
    return n


def bq_version() -> int:
    return int(lib().bq_version())


# --- small conveniences that only allocate (no arithmetic) -------------------------------------

def alloc_plan(theta, n: int, heads: int = 1, stream=None):
    """Allocate a plan buffer with torch and fill it from `theta` (float32 device tensor)."""
    import torch

    nbytes = bq_plan_bytes(n, heads)
    if nbytes == 0:
        raise BqError(2, f"invalid plan shape n={n} heads={heads}")
    plan = torch.empty(nbytes, dtype=torch.uint8, device=theta.device)
    bq_plan_build(theta, n, heads, plan, stream)
    return plan


def alloc_quant_outputs(rows: int, n: int, heads: int, bits: int, group: int, scale_dtype: str, device):
    import torch

    codes = torch.empty((rows, n * heads * bits // 8), dtype=torch.uint8, device=device)
    sd = torch.float16 if scale_dtype == "f16" else torch.float32
    scales = torch.empty((rows, n * heads // group), dtype=sd, device=device)
    return codes, scales


def make_quant(bits: int, group: int, scale_dtype: str) -> bq_quant:
    q = bq_quant()
    q.bits, q.group, q.scale_dtype = bits, group, DTYPE_CODES[scale_dtype]
    return q
