"""ctypes binding of libgsi.so: argument marshalling only.

Function names, argument order and meaning follow ``include/gsi.h``.  Tensors are torch CUDA
(ROCm) tensors used purely as device memory; their ``data_ptr()`` and the current torch stream
handle are what crosses the boundary.  Every step of the path runs inside the library's HIP
kernels; there is no fallback: if ``libgsi.so`` is missing, importing this module raises.
"""
from __future__ import annotations

import ctypes
import functools
import os
import threading
from typing import List, Optional, Sequence, Tuple

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libgsi.so")

GSI_OK = 0
GSI_ERR_NULL, GSI_ERR_SHAPE, GSI_ERR_DTYPE, GSI_ERR_ALIGN, GSI_ERR_WORKSPACE, GSI_ERR_HIP = -1, -2, -3, -4, -5, -6
GSI_F32, GSI_BF16 = 0, 1
INPUT_SLOW_PATH_WX = 1  # gsi_input_desc.flags: fired tokens get y = W x (Algorithm 1, line 7)
INPUT_FUSED_KERNEL = 2  # gsi_input_desc.flags: single-token calls take the fused kernel (one launch, basis read once)
INPUT_GATE_SINGLE_PASS = 4  # gsi_input_desc.flags: residual ratio from |x|^2 - |c|^2 + c^T E c, E = U^T U - I (`gram`)
MAP_IMAGE_FP8 = 1  # gsi_map_desc.flags: M holds E4M3 codes, M_scale the row scales (single-token calls)
CALL_BUILD_IMAGE, CALL_PROJECT, CALL_GATE, CALL_GATED_LINEAR, CALL_DENSE_LINEAR, CALL_LAYER_STACK = range(6)

EXPORTS = (
    "gsi_build_image", "gsi_build_gram", "gsi_extend_basis", "gsi_extend_basis_workspace_bytes", "gsi_extend_many", "gsi_extend_many_workspace_bytes", "gsi_quantize_image_fp8", "gsi_project", "gsi_gate", "gsi_gated_linear", "gsi_dense_linear",
    "gsi_layer_stack",
    "gsi_layer_stack_static", "gsi_layer_stack_timed", "gsi_dense_stack",
    "gsi_stack_plan_bytes", "gsi_stack_plan_build", "gsi_stack_plan_run",
    "gsi_workspace_bytes", "gsi_layer_stack_workspace_bytes", "gsi_dense_stack_workspace_bytes", "gsi_last_error",
    "gsi_fused_timeouts",
    "gsi_version",
)


class GsiError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"libgsi error {code}: {msg}")
        self.code = code


class InputDesc(ctypes.Structure):
    _fields_ = [
        ("U", ctypes.c_void_p), ("X", ctypes.c_void_p),
        ("d", ctypes.c_int64), ("k", ctypes.c_int64),
        ("udtype", ctypes.c_int32), ("xdtype", ctypes.c_int32),
        ("C", ctypes.c_void_p), ("R", ctypes.c_void_p),
        ("rnorm", ctypes.c_void_p), ("xnorm", ctypes.c_void_p),
        ("mask", ctypes.c_void_p), ("fired_idx", ctypes.c_void_p), ("n_fired", ctypes.c_void_p),
        ("src_map", ctypes.c_int32), ("flags", ctypes.c_int32),
        ("gram", ctypes.c_void_p),
    ]


class ExtendMap(ctypes.Structure):
    _fields_ = [("W", ctypes.c_void_p), ("M", ctypes.c_void_p), ("m", ctypes.c_int64)]


class ExtendDesc(ctypes.Structure):
    _fields_ = [
        ("U", ctypes.c_void_p), ("d", ctypes.c_int64), ("K", ctypes.c_int64), ("udtype", ctypes.c_int32),
        ("n_maps", ctypes.c_int32), ("k_cur", ctypes.c_void_p), ("R", ctypes.c_void_p), ("rnorm", ctypes.c_void_p),
        ("xnorm", ctypes.c_void_p), ("maps", ctypes.POINTER(ExtendMap)), ("gram", ctypes.c_void_p),
        ("extended", ctypes.c_void_p),
    ]


class StackPlan(ctypes.Structure):
    _fields_ = [("opaque", ctypes.c_uint64 * 24)]


class MapDesc(ctypes.Structure):
    _fields_ = [
        ("W", ctypes.c_void_p), ("M", ctypes.c_void_p), ("Y", ctypes.c_void_p),
        ("m", ctypes.c_int64), ("wdtype", ctypes.c_int32), ("input_id", ctypes.c_int32),
        ("M_scale", ctypes.c_void_p), ("flags", ctypes.c_int32), ("reserved", ctypes.c_int32),
    ]


def _load() -> ctypes.CDLL:
    if not os.path.exists(LIB_PATH):
        raise ImportError(
            f"{LIB_PATH} is missing: build it with `python -m paper_2605_03109_amd.build` "
            "(there is no CPU or PyTorch fallback for the HIP path)"
        )
    lib = ctypes.CDLL(LIB_PATH)
    vp, i64, i32, sz, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t, ctypes.c_float
    lib.gsi_build_image.argtypes = [vp, vp, vp, i64, i64, i64, i32, vp, sz, vp]
    lib.gsi_quantize_image_fp8.argtypes = [vp, i32, i64, i64, vp, vp, vp]
    lib.gsi_build_gram.argtypes = [vp, i64, i64, i32, vp, vp]
    lib.gsi_extend_basis.argtypes = [vp, i64, i64, i32, vp, vp, vp, vp, f32, ctypes.POINTER(ExtendMap), ctypes.c_int32,
                                     vp, vp, vp, sz, vp]
    lib.gsi_extend_basis.restype = ctypes.c_int
    lib.gsi_extend_basis_workspace_bytes.argtypes = [i64, i64]
    lib.gsi_extend_basis_workspace_bytes.restype = sz
    lib.gsi_extend_many.argtypes = [ctypes.POINTER(ExtendDesc), i32, f32, vp, sz, vp]
    lib.gsi_extend_many.restype = ctypes.c_int
    lib.gsi_extend_many_workspace_bytes.argtypes = [ctypes.POINTER(ExtendDesc), i32]
    lib.gsi_extend_many_workspace_bytes.restype = sz
    lib.gsi_project.argtypes = [vp, vp, i64, i64, i64, i32, i32, vp, vp, vp, vp, vp, sz, vp]
    lib.gsi_gate.argtypes = [vp, vp, i64, f32, vp, vp, vp, vp]
    lib.gsi_gated_linear.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i32, vp, i32, vp, sz, vp]
    lib.gsi_dense_linear.argtypes = [vp, vp, i64, i64, i64, i32, i32, vp, vp, sz, vp]
    lib.gsi_layer_stack.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32, ctypes.POINTER(InputDesc),
                                    ctypes.c_int32, i64, f32, vp, sz, vp]
    lib.gsi_layer_stack_static.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32, ctypes.POINTER(InputDesc),
                                           ctypes.c_int32, i64, f32, vp]
    lib.gsi_layer_stack_static.restype = ctypes.c_int
    lib.gsi_layer_stack_timed.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32, ctypes.POINTER(InputDesc),
                                          ctypes.c_int32, i64, f32, vp, sz, vp, i32, i32, vp, vp]
    lib.gsi_stack_plan_bytes.argtypes = [ctypes.c_int32, ctypes.c_int32]
    lib.gsi_stack_plan_bytes.restype = sz
    lib.gsi_stack_plan_build.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32, ctypes.POINTER(InputDesc), ctypes.c_int32,
                                         vp, sz, vp, sz, ctypes.POINTER(StackPlan), vp]
    lib.gsi_stack_plan_build.restype = ctypes.c_int
    lib.gsi_stack_plan_run.argtypes = [ctypes.POINTER(StackPlan), f32, vp]
    lib.gsi_stack_plan_run.restype = ctypes.c_int
    lib.gsi_dense_stack.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32, ctypes.POINTER(InputDesc),
                                    ctypes.c_int32, i64, vp, sz, vp]
    lib.gsi_workspace_bytes.argtypes = [i32, i64, i64, i64, i64]
    lib.gsi_workspace_bytes.restype = sz
    lib.gsi_layer_stack_workspace_bytes.argtypes = [ctypes.POINTER(MapDesc), ctypes.c_int32,
                                                    ctypes.POINTER(InputDesc), ctypes.c_int32, i64]
    lib.gsi_layer_stack_workspace_bytes.restype = sz
    lib.gsi_dense_stack_workspace_bytes.argtypes = lib.gsi_layer_stack_workspace_bytes.argtypes
    lib.gsi_dense_stack_workspace_bytes.restype = sz
    lib.gsi_fused_timeouts.argtypes = [ctypes.POINTER(ctypes.c_uint32)]
    lib.gsi_fused_timeouts.restype = ctypes.c_int
    lib.gsi_last_error.restype = ctypes.c_char_p
    lib.gsi_version.restype = ctypes.c_int
    for name in ("gsi_build_image", "gsi_build_gram", "gsi_quantize_image_fp8", "gsi_project", "gsi_gate", "gsi_gated_linear", "gsi_dense_linear",
                 "gsi_layer_stack", "gsi_layer_stack_timed", "gsi_dense_stack"):
        getattr(lib, name).restype = ctypes.c_int
    return lib


lib = _load()


def _check(rc: int) -> None:
    if rc != GSI_OK:
        raise GsiError(rc, lib.gsi_last_error().decode())


def last_error() -> str:
    return lib.gsi_last_error().decode()


def version() -> int:
    return lib.gsi_version()


def fused_timeouts() -> int:
    """Bounded waits of fused-kernel launches that expired on the current device (0 in normal operation)."""
    n = ctypes.c_uint32(0)
    _check(lib.gsi_fused_timeouts(ctypes.byref(n)))
    return int(n.value)


# ----------------------------------------------------------------------------------------------
# marshalling helpers
# ----------------------------------------------------------------------------------------------
def dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return GSI_F32
    if t.dtype == torch.bfloat16:
        return GSI_BF16
    raise TypeError(f"unsupported tensor dtype {t.dtype}")


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("libgsi takes device tensors only")
    if not t.is_contiguous():
        raise ValueError("libgsi takes contiguous row-major tensors only")
    return t.data_ptr()


# The current device and the raw handle of its current stream without a Stream object and an initialisation check per
# call, where this torch has the functions for it: three calls of one fp32 map, one token, are bound by the host (passes
# back to back: 38.6 us with the object, 32.5 us without)
_get_device = getattr(torch._C, "_cuda_getDevice", None) or torch.cuda.current_device
_raw_stream = (getattr(torch._C, "_cuda_getCurrentRawStream", None)
               or (lambda device: torch.cuda.current_stream(device).cuda_stream))


def _device() -> int:
    return _get_device() if torch.cuda.is_initialized() else torch.cuda.current_device()


def _stream(stream=None) -> int:
    return _raw_stream(_device()) if stream is None else stream.cuda_stream


def to_device(a: np.ndarray, dtype: str, device="cuda") -> torch.Tensor:
    """Stored operand (fp32 array or uint16 bf16 bit patterns) -> device tensor, bit for bit."""
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(device)
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(device)


def bits_of(t: torch.Tensor) -> np.ndarray:
    """Device tensor -> host array in the storage convention of the workload module."""
    if t.dtype == torch.bfloat16:
        return t.detach().cpu().contiguous().view(torch.int16).numpy().view(np.uint16)
    return t.detach().cpu().numpy()


_WS_KEPT = 8                  # buffers that a thread keeps
_ws_local = threading.local()  # {(device, raw stream): buffer} in order of use, one table per thread


def workspace(nbytes: int, device=None, stream=None) -> Optional[torch.Tensor]:
    """A device byte buffer of at least ``nbytes`` for a call on ``stream`` (None: the current one).

    A call's kernels leave partial sums and completion counters there, so calls that may overlap never share one: every
    thread keeps a buffer per stream, allocated on that stream (what an outgrown or dropped buffer gives back is
    used again behind the stream's work only).  Under capture the buffer is the graph's and is not kept."""
    if nbytes == 0:
        return None
    if stream is not None:
        if not isinstance(stream, torch.cuda.Stream):
            stream = torch.cuda.ExternalStream(stream.cuda_stream)
        with torch.cuda.stream(stream):
            return workspace(nbytes, device)
    dev = _device() if device is None else torch.device(device).index or 0
    if torch.cuda.is_current_stream_capturing():
        return torch.empty(nbytes, dtype=torch.uint8, device=f"cuda:{dev}")
    kept, key = _ws_local.__dict__, (dev, _raw_stream(dev))
    have = kept.pop(key, None)
    if have is None or have.numel() < nbytes:
        have = torch.empty(max(nbytes, 1 << 20), dtype=torch.uint8, device=f"cuda:{dev}")
        while len(kept) >= _WS_KEPT:
            del kept[next(iter(kept))]
    kept[key] = have
    return have


@functools.lru_cache(maxsize=4096, typed=True)  # (of the sizes alone; 0.15 us instead of 1.1 for a known call; 4096.0 is refused behind 4096 too)
def workspace_bytes(which: int, m: int = 0, d: int = 0, k: int = 0, B: int = 0) -> int:
    return int(lib.gsi_workspace_bytes(which, m, d, k, B))


def _ws_args(ws: Optional[torch.Tensor], need: int, stream=None):
    """(pointer, bytes, the tensor that the caller holds until its call is enqueued)"""
    if ws is None:
        ws = workspace(need, stream=stream)
    return (None, 0, None) if ws is None else (ws.data_ptr(), ws.numel() * ws.element_size(), ws)


# ----------------------------------------------------------------------------------------------
# entry points (same names as the C ABI, minus the prefix)
# ----------------------------------------------------------------------------------------------
def build_image(W: torch.Tensor, U: torch.Tensor, M: Optional[torch.Tensor] = None, ws=None, stream=None):
    m, d = W.shape
    d2, k = U.shape
    if d2 != d or W.dtype != U.dtype:
        raise ValueError("W[m,d] and U[d,k] must agree in d and dtype")
    if M is None:
        M = torch.empty((m, k), dtype=W.dtype, device=W.device)
    wsp, wsn, held = _ws_args(ws, workspace_bytes(CALL_BUILD_IMAGE, m, d, k, 0), stream)
    _check(lib.gsi_build_image(_ptr(W), _ptr(U), _ptr(M), m, d, k, dtype_code(W), wsp, wsn, _stream(stream)))
    return M


def build_gram(U: torch.Tensor, E: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """E[k,k] (fp32) = U^T U - I of a stored basis U[d,k]."""
    d, k = U.shape
    E = torch.empty((k, k), dtype=torch.float32, device=U.device) if E is None else E
    _check(lib.gsi_build_gram(_ptr(U), d, k, dtype_code(U), _ptr(E), _stream(stream)))
    return E


def extend_basis(U: torch.Tensor, k_cur: torch.Tensor, R: torch.Tensor, rnorm: torch.Tensor, xnorm: torch.Tensor,
                 tau: float, maps: Sequence[Tuple[torch.Tensor, torch.Tensor]] = (), gram: Optional[torch.Tensor] = None,
                 extended: Optional[torch.Tensor] = None, ws=None, stream=None) -> torch.Tensor:
    """One rank-1 extension step of the basis array U[d,K] (in place); maps: (W[m,d], M[m,K]) pairs whose column
    k_cur is appended.  Returns the device flag ``extended`` (int32[1])."""
    d, K = U.shape
    extended = torch.zeros((1,), dtype=torch.int32, device=U.device) if extended is None else extended
    em = (ExtendMap * max(len(maps), 1))()
    for j, (W, M) in enumerate(maps):
        if W.dtype != U.dtype or M.dtype != U.dtype or tuple(M.shape) != (W.shape[0], K) or W.shape[1] != d:
            raise ValueError("maps must be (W[m,d], M[m,K]) in the basis' dtype")
        em[j].W, em[j].M, em[j].m = _ptr(W), _ptr(M), W.shape[0]
    wsp, wsn, held = _ws_args(ws, int(lib.gsi_extend_basis_workspace_bytes(d, K)), stream)
    _check(lib.gsi_extend_basis(_ptr(U), d, K, dtype_code(U), _ptr(k_cur), _ptr(R), _ptr(rnorm), _ptr(xnorm), float(tau),
                                em, len(maps), _ptr(gram), _ptr(extended), wsp, wsn, _stream(stream)))
    return extended


class ExtendSet:
    """The bases of a model that see every token (gsi_extend_many): descriptors marshalled once, one call per token.

    ``bases``: list of dicts {U[d,K], k_cur, R[d], rnorm, xnorm, maps: [(W[m,d], M[m,K]), ...]} (+ gram, + extended);
    every tensor is kept alive by the set."""

    def __init__(self, bases: Sequence[dict]):
        self.bases = list(bases)
        n = len(self.bases)
        self._desc = (ExtendDesc * max(n, 1))()
        self._maps = []
        for i, b in enumerate(self.bases):
            U = b["U"]
            d, K = U.shape
            maps = list(b.get("maps", ()))
            em = (ExtendMap * max(len(maps), 1))()
            for j, (W, M) in enumerate(maps):
                if W.dtype != U.dtype or M.dtype != U.dtype or tuple(M.shape) != (W.shape[0], K) or W.shape[1] != d:
                    raise ValueError("maps must be (W[m,d], M[m,K]) in the basis' dtype")
                em[j].W, em[j].M, em[j].m = _ptr(W), _ptr(M), W.shape[0]
            self._maps.append(em)
            if b.get("extended") is None:
                b["extended"] = torch.zeros((1,), dtype=torch.int32, device=U.device)
            e = self._desc[i]
            e.U, e.d, e.K, e.udtype, e.n_maps = _ptr(U), d, K, dtype_code(U), len(maps)
            e.k_cur, e.R, e.rnorm, e.xnorm = _ptr(b["k_cur"]), _ptr(b["R"]), _ptr(b["rnorm"]), _ptr(b["xnorm"])
            e.maps = em
            e.gram, e.extended = _ptr(b.get("gram")), _ptr(b["extended"])
        self.n = n
        need = int(lib.gsi_extend_many_workspace_bytes(self._desc, n)) if n else 0
        dev = self.bases[0]["U"].device if n else "cuda"
        self.ws = torch.empty((need + 256,), dtype=torch.uint8, device=dev)
        off = (-self.ws.data_ptr()) % 256
        self._wsp, self._wsn = self.ws.data_ptr() + off, need

    def step(self, tau: float, stream=None) -> None:
        """One extension step of every basis on the token whose R, rnorm, xnorm the descriptors point at."""
        _check(lib.gsi_extend_many(self._desc, self.n, float(tau), self._wsp, self._wsn, _stream(stream)))


def quantize_image_fp8(M: torch.Tensor, M8: Optional[torch.Tensor] = None, scale: Optional[torch.Tensor] = None,
                       stream=None):
    """E4M3 codes M8[m,k] (uint8) and power-of-two row scales scale[m] (fp32) of a stored image M[m,k]."""
    m, k = M.shape
    M8 = torch.empty((m, k), dtype=torch.uint8, device=M.device) if M8 is None else M8
    scale = torch.empty((m,), dtype=torch.float32, device=M.device) if scale is None else scale
    _check(lib.gsi_quantize_image_fp8(_ptr(M), dtype_code(M), m, k, _ptr(M8), _ptr(scale), _stream(stream)))
    return M8, scale


def project(U: torch.Tensor, X: torch.Tensor, C=None, R=None, rnorm=None, xnorm=None, ws=None, stream=None):
    d, k = U.shape
    B, d2 = X.shape
    if d2 != d:
        raise ValueError("U[d,k] and X[B,d] must agree in d")
    f32 = dict(dtype=torch.float32, device=U.device)
    C = torch.empty((B, k), **f32) if C is None else C
    R = torch.empty((B, d), **f32) if R is None else R
    rnorm = torch.empty((B,), **f32) if rnorm is None else rnorm
    xnorm = torch.empty((B,), **f32) if xnorm is None else xnorm
    wsp, wsn, held = _ws_args(ws, workspace_bytes(CALL_PROJECT, 0, d, k, B), stream)
    _check(lib.gsi_project(_ptr(U), _ptr(X), d, k, B, dtype_code(U), dtype_code(X), _ptr(C), _ptr(R), _ptr(rnorm),
                           _ptr(xnorm), wsp, wsn, _stream(stream)))
    return C, R, rnorm, xnorm


def gate(rnorm: torch.Tensor, xnorm: torch.Tensor, eps: float, mask=None, fired_idx=None, n_fired=None, stream=None):
    B = rnorm.shape[0]
    dev = rnorm.device
    mask = torch.empty((B,), dtype=torch.uint8, device=dev) if mask is None else mask
    fired_idx = torch.empty((max(B, 1),), dtype=torch.int32, device=dev) if fired_idx is None else fired_idx
    n_fired = torch.empty((1,), dtype=torch.int32, device=dev) if n_fired is None else n_fired
    _check(lib.gsi_gate(_ptr(rnorm), _ptr(xnorm), B, float(eps), _ptr(mask), _ptr(fired_idx), _ptr(n_fired),
                        _stream(stream)))
    return mask, fired_idx, n_fired


def gated_linear(W, M, C, R, fired_idx, n_fired, Y=None, ws=None, stream=None):
    m, d = W.shape
    k = M.shape[1]
    B = C.shape[0]
    if M.shape[0] != m or C.shape[1] != k or tuple(R.shape) != (B, d) or M.dtype != W.dtype:
        raise ValueError("inconsistent shapes/dtypes for gated_linear")
    Y = torch.empty((B, m), dtype=torch.float32, device=W.device) if Y is None else Y
    wsp, wsn, held = _ws_args(ws, workspace_bytes(CALL_GATED_LINEAR, m, d, k, B), stream)
    _check(lib.gsi_gated_linear(_ptr(W), _ptr(M), _ptr(C), _ptr(R), _ptr(fired_idx), _ptr(n_fired), m, d, k, B,
                                dtype_code(W), _ptr(Y), GSI_F32, wsp, wsn, _stream(stream)))
    return Y


def dense_linear(W, X, Y=None, ws=None, stream=None):
    m, d = W.shape
    B = X.shape[0]
    if X.shape[1] != d:
        raise ValueError("W[m,d] and X[B,d] must agree in d")
    Y = torch.empty((B, m), dtype=torch.float32, device=W.device) if Y is None else Y
    wsp, wsn, held = _ws_args(ws, workspace_bytes(CALL_DENSE_LINEAR, m, d, 0, B), stream)
    _check(lib.gsi_dense_linear(_ptr(W), _ptr(X), m, d, B, dtype_code(W), dtype_code(X), _ptr(Y), wsp, wsn,
                                _stream(stream)))
    return Y


class LayerStack:
    """Host descriptor tables for ``gsi_layer_stack`` plus the device buffers they point to.

    ``inputs``: list of dicts {U, X (tensor [B,d]) or src_map} (+ flags, + gram: the tensor of ``build_gram``); ``maps``: list of dicts
    {W, M, input_id} (+ M_scale when M holds the E4M3 codes of ``quantize_image_fp8``).  Output buffers are allocated here (torch = device memory only) and exposed as
    attributes; ``run()`` is a single call into the library.
    """

    def __init__(self, inputs: Sequence[dict], maps: Sequence[dict], B: int, eps: float):
        self.B, self.eps = int(B), float(eps)
        dev = maps[0]["W"].device
        f32 = dict(dtype=torch.float32, device=dev)
        self.maps_t: List[dict] = []
        self.inputs_t: List[dict] = []
        for mp in maps:
            m = mp["W"].shape[0]
            Y = mp.get("Y")
            Y = torch.zeros((B, m), **f32) if Y is None else Y
            self.maps_t.append({"W": mp["W"], "M": mp["M"], "Y": Y, "input_id": int(mp["input_id"]),
                                "M_scale": mp.get("M_scale")})
        for inp in inputs:
            U = inp["U"]
            d, k = U.shape
            src = int(inp.get("src_map", -1))
            X = self.maps_t[src]["Y"] if src >= 0 else inp["X"]
            self.inputs_t.append({
                "U": U, "X": X, "src_map": src, "flags": int(inp.get("flags", 0)), "gram": inp.get("gram"),
                "C": torch.zeros((B, k), **f32), "R": torch.zeros((B, d), **f32),
                "rnorm": torch.zeros((B,), **f32), "xnorm": torch.zeros((B,), **f32),
                "mask": torch.zeros((B,), dtype=torch.uint8, device=dev),
                "fired_idx": torch.zeros((max(B, 1),), dtype=torch.int32, device=dev),
                "n_fired": torch.zeros((1,), dtype=torch.int32, device=dev),
            })
        self._in = (InputDesc * len(self.inputs_t))()
        self._mp = (MapDesc * len(self.maps_t))()
        self.ws = torch.empty(256, dtype=torch.uint8, device=dev)
        self.refresh()

    def refresh(self, token_offset: int = 0, B: Optional[int] = None) -> None:
        """(Re)write the descriptor tables; ``token_offset`` selects rows [offset, offset+B) of every buffer."""
        B = self.B if B is None else B
        self.cur_B = B
        o = token_offset
        for i, t in enumerate(self.inputs_t):
            d, k = t["U"].shape
            e = self._in[i]
            e.U, e.d, e.k = _ptr(t["U"]), d, k
            e.X = _ptr(t["X"]) + o * d * t["X"].element_size()
            e.udtype, e.xdtype = dtype_code(t["U"]), dtype_code(t["X"])
            e.C = _ptr(t["C"]) + o * k * 4
            e.R = _ptr(t["R"]) + o * d * 4
            e.rnorm = _ptr(t["rnorm"]) + o * 4
            e.xnorm = _ptr(t["xnorm"]) + o * 4
            e.mask = _ptr(t["mask"]) + o
            e.fired_idx = _ptr(t["fired_idx"])
            e.n_fired = _ptr(t["n_fired"])
            e.src_map, e.flags = t["src_map"], t["flags"]
            e.gram = _ptr(t["gram"])
        for j, t in enumerate(self.maps_t):
            m = t["W"].shape[0]
            e = self._mp[j]
            e.W, e.M, e.m = _ptr(t["W"]), _ptr(t["M"]), m
            e.Y = _ptr(t["Y"]) + o * m * 4
            e.wdtype, e.input_id = dtype_code(t["W"]), t["input_id"]
            e.M_scale = _ptr(t["M_scale"])
            e.flags, e.reserved = (MAP_IMAGE_FP8 if t["M_scale"] is not None else 0), 0
        need = max(int(fn(self._mp, len(self.maps_t), self._in, len(self.inputs_t), B))
                   for fn in (lib.gsi_layer_stack_workspace_bytes, lib.gsi_dense_stack_workspace_bytes))
        if need > self.ws.numel():  # the workspace depends on the token count of the call
            self.ws = torch.empty(need, dtype=torch.uint8, device=self.ws.device)

    def run(self, stream=None) -> None:
        _check(lib.gsi_layer_stack(self._mp, len(self.maps_t), self._in, len(self.inputs_t), self.cur_B, self.eps,
                                   self.ws.data_ptr(), self.ws.numel(), _stream(stream)))

    def run_static(self, stream=None) -> None:
        """As run(), with the scratch memory in the library's static device array (no workspace argument)."""
        _check(lib.gsi_layer_stack_static(self._mp, len(self.maps_t), self._in, len(self.inputs_t), self.cur_B, self.eps,
                                          _stream(stream)))

    def run_timed(self, ev_begin: int, ev_end: int, stream=None, which: int = 0, index: int = 0) -> None:
        """As run(), with raw hipEvent_t handles that take the dispatch timestamps of one launch of the call
        (which: 0 = staged projection kernel, 1 = weight streaming; index: which launch of that kind)."""
        _check(lib.gsi_layer_stack_timed(self._mp, len(self.maps_t), self._in, len(self.inputs_t), self.cur_B,
                                         self.eps, self.ws.data_ptr(), self.ws.numel(), _stream(stream), which, index,
                                         ev_begin, ev_end))

    def build_plan(self, stream=None):
        """Marshal the current descriptor tables (as refresh() left them, one token per call) once: returns
        (plan, plan_mem); plan_mem and self.ws must be kept alive while the plan is used."""
        nbytes = int(lib.gsi_stack_plan_bytes(len(self.maps_t), len(self.inputs_t)))
        mem = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=self.ws.device)
        plan = StackPlan()
        _check(lib.gsi_stack_plan_build(self._mp, len(self.maps_t), self._in, len(self.inputs_t), self.ws.data_ptr(),
                                        self.ws.numel(), mem.data_ptr(), mem.numel(), ctypes.byref(plan), _stream(stream)))
        return plan, mem

    def run_plan(self, plan, stream=None) -> None:
        _check(lib.gsi_stack_plan_run(ctypes.byref(plan), self.eps, _stream(stream)))

    def run_dense(self, stream=None) -> None:
        """The dense baseline Y = W X over the same descriptor tables (one launch for all maps)."""
        _check(lib.gsi_dense_stack(self._mp, len(self.maps_t), self._in, len(self.inputs_t), self.cur_B,
                                   self.ws.data_ptr(), self.ws.numel(), _stream(stream)))


def layer_stack(inputs: Sequence[dict], maps: Sequence[dict], B: int, eps: float, stream=None) -> LayerStack:
    st = LayerStack(inputs, maps, B, eps)
    st.run(stream)
    return st
