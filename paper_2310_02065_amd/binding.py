"""ctypes binding of libvenom.so: argument marshalling only.

Every step of the path (compression, packing, the product) runs in the library's HIP kernels;
PyTorch supplies device memory and streams.  There is no CPU fallback: if the shared library has
not been built, `lib()` raises.

Every call takes a `stream` (default: the current one).  Tensors made for the caller -- results, a handle's workspace --
belong to the current stream all the same: where another one is passed, it is the caller who has it wait for the current
stream and keeps them until their work is done, as with any tensor that is used on a second stream.
"""
from __future__ import annotations

import ctypes
import os
import threading
from ctypes import POINTER, byref, c_char_p, c_int, c_int64, c_size_t, c_void_p
from threading import get_ident

import torch

# What torch.cuda's functions call, without their wrappers (each costs a few tenths of a microsecond per library call).
_current_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_current_device = getattr(torch._C, "_cuda_getDevice", torch.cuda.current_device)
_is_current_stream_capturing = getattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: False)

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libvenom.so")

VENOM_OK = 0
STATUS_NAMES = {
    0: "VENOM_OK", 1: "VENOM_ERR_INVALID_ARG", 2: "VENOM_ERR_SHAPE", 3: "VENOM_ERR_UNSUPPORTED",
    4: "VENOM_ERR_MASK_COLS", 5: "VENOM_ERR_MASK_ROW", 6: "VENOM_ERR_WORKSPACE", 7: "VENOM_ERR_HIP",
}
(VENOM_ERR_INVALID_ARG, VENOM_ERR_SHAPE, VENOM_ERR_UNSUPPORTED, VENOM_ERR_MASK_COLS, VENOM_ERR_MASK_ROW,
 VENOM_ERR_WORKSPACE, VENOM_ERR_HIP) = range(1, 8)

# every symbol include/venom.h declares
EXPORTS = ("venom_workspace_bytes", "venom_prune", "venom_compress", "venom_import", "venom_export", "venom_decompress",
           "venom_spmm", "venom_spmm_variant", "venom_spmm_bias_act", "venom_linear_scratch_bytes", "venom_linear",
           "venom_linear_static_max_bytes", "venom_linear_static", "venom_energy", "venom_probe_smfmac_rate",
           "venom_spmm_variant_count", "venom_spmm_variant_name",
           "venom_get_info", "venom_destroy", "venom_status_string")


class Violation(ctypes.Structure):
    _fields_ = [("block_row", c_int64), ("group", c_int64), ("row", c_int64)]


class VenomError(RuntimeError):
    def __init__(self, status, where, violation=None):
        self.status = status
        self.violation = violation
        msg = f"{where}: {STATUS_NAMES.get(status, status)}"
        if violation is not None:
            msg += f" at (block_row, group, row)={violation}"
        super().__init__(msg)


_lib = None


def lib() -> ctypes.CDLL:
    """Loads the HIP library; raises if it is missing (there is no other implementation)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} not found: build it first (python -m paper_2310_02065_amd.build)")
    L = ctypes.CDLL(LIB_PATH)
    L.venom_workspace_bytes.argtypes = [c_int64, c_int64, c_int, c_int, c_int, POINTER(c_size_t)]
    L.venom_compress.argtypes = [c_void_p, c_int64, c_void_p, c_int64, c_int64, c_int64, c_int, c_int, c_int,
                                 c_void_p, c_size_t, c_void_p, POINTER(c_void_p), POINTER(Violation)]
    L.venom_prune.argtypes = [c_void_p, c_int64, c_int64, c_int64, c_int, c_int, c_int, c_void_p, c_int64, c_void_p,
                              c_void_p, c_void_p]
    L.venom_import.argtypes = [c_void_p, c_void_p, c_void_p, c_int64, c_int64, c_int, c_int, c_int, c_void_p,
                               c_size_t, c_void_p, POINTER(c_void_p)]
    L.venom_export.argtypes = [c_void_p, c_void_p, c_void_p, c_void_p, c_void_p]
    L.venom_decompress.argtypes = [c_void_p, c_void_p, c_int64, c_void_p]
    L.venom_spmm.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int64, c_int, c_void_p]
    L.venom_spmm_variant.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int64, c_int, c_int, c_void_p]
    L.venom_spmm_bias_act.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int, c_void_p, c_int64, c_int,
                                      c_int, c_void_p]
    L.venom_linear_scratch_bytes.argtypes = [c_void_p, c_int64, POINTER(c_size_t)]
    L.venom_linear.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int, c_void_p, c_int64, c_int, c_void_p,
                               c_size_t, c_void_p]
    L.venom_linear_static_max_bytes.argtypes = []
    L.venom_linear_static_max_bytes.restype = c_size_t
    L.venom_linear_static.argtypes = [c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int, c_void_p, c_int64, c_int,
                                      c_void_p]
    L.venom_energy.argtypes = [c_void_p, c_void_p, c_int64, POINTER(ctypes.c_double), c_void_p]
    L.venom_probe_smfmac_rate.argtypes = [c_int, c_void_p, c_void_p]
    L.venom_spmm_variant_count.argtypes = []
    L.venom_spmm_variant_name.argtypes = [c_int]
    L.venom_spmm_variant_name.restype = c_char_p
    L.venom_get_info.argtypes = [c_void_p, POINTER(c_int64), POINTER(c_int64), POINTER(c_int), POINTER(c_int),
                                 POINTER(c_int)]
    L.venom_destroy.argtypes = [c_void_p]
    L.venom_destroy.restype = None
    L.venom_status_string.argtypes = [c_int]
    L.venom_status_string.restype = c_char_p
    for name in ("venom_workspace_bytes", "venom_prune", "venom_compress", "venom_import", "venom_export", "venom_decompress",
                 "venom_spmm", "venom_spmm_variant", "venom_spmm_bias_act", "venom_linear_scratch_bytes", "venom_linear",
                 "venom_linear_static", "venom_energy", "venom_probe_smfmac_rate", "venom_spmm_variant_count", "venom_get_info"):
        getattr(L, name).restype = c_int
    _lib = L
    return L


def _stream_ptr(stream=None):
    """The stream's handle as an integer; the current device's current stream by default.  (Asked for by itself it takes
    0.2 us; torch.cuda.current_stream() makes an object of it first, 1.5 us.)"""
    if stream is not None:
        return stream.cuda_stream
    if _current_raw_stream is None:
        return torch.cuda.current_stream().cuda_stream
    return _current_raw_stream(_current_device())            # (there are CUDA tensors, so CUDA is initialised)


def _ptr(t):
    return t.data_ptr() if t is not None else None


def venom_workspace_bytes(R, K, V, N, M) -> int:
    n = c_size_t(0)
    st = lib().venom_workspace_bytes(R, K, V, N, M, byref(n))
    if st != VENOM_OK:
        raise VenomError(st, "venom_workspace_bytes")
    return n.value


class Handle:
    """Owns the workspace tensor and the host-side handle of one compressed matrix."""

    def __init__(self, ptr, workspace, R, K, V, N, M):
        self.ptr, self.workspace = ptr, workspace
        self.R, self.K, self.V, self.N, self.M = R, K, V, N, M

    @property
    def G(self):
        return self.K // self.M

    def close(self):
        if self.ptr:
            lib().venom_destroy(self.ptr)
            self.ptr = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def _workspace(R, K, V, N, M, device):
    nbytes = venom_workspace_bytes(R, K, V, N, M)
    ws = torch.empty(max(nbytes, 256) + 256, dtype=torch.uint8, device=device)
    off = (-ws.data_ptr()) % 256
    return ws, ws[off:off + max(nbytes, 256)], nbytes


def venom_compress(A, mask, V, N, M, stream=None) -> Handle:
    """A: R x K float16 CUDA tensor (row stride lda), mask: R x K uint8 CUDA tensor."""
    assert A.is_cuda and mask.is_cuda and A.dtype == torch.float16 and mask.dtype in (torch.uint8, torch.bool)
    assert A.dim() == 2 and mask.shape == A.shape and A.stride(1) == 1 and mask.stride(1) == 1
    R, K = A.shape
    ws_owner, ws, nbytes = _workspace(R, K, V, N, M, A.device)
    out = c_void_p(0)
    viol = Violation(-1, -1, -1)
    st = lib().venom_compress(_ptr(A), A.stride(0) if R > 1 else max(K, A.stride(0)), _ptr(mask),
                              mask.stride(0) if R > 1 else max(K, mask.stride(0)), R, K, V, N, M, _ptr(ws), nbytes,
                              _stream_ptr(stream), byref(out), byref(viol))
    if st != VENOM_OK:
        v = (viol.block_row, viol.group, viol.row) if st in (VENOM_ERR_MASK_COLS, VENOM_ERR_MASK_ROW) else None
        raise VenomError(st, "venom_compress", v)
    h = Handle(out, ws, R, K, V, N, M)
    h._owner = ws_owner
    return h


def venom_prune(A, V, N, M, stream=None):
    """Magnitude pruning of A (R x K float16 CUDA tensor) to V:N:M.  Returns (mask uint8 R x K,
    kept_mass int64 [R/V], total_mass int64 [R/V]); the masses are exact integers in units of 2^-24."""
    assert A.is_cuda and A.dtype == torch.float16 and A.dim() == 2 and A.stride(1) == 1
    R, K = A.shape
    mask = torch.empty((R, K), dtype=torch.uint8, device=A.device)
    nb = max(R // V, 1) if V > 0 else 1
    kept = torch.empty(nb, dtype=torch.int64, device=A.device)
    total = torch.empty(nb, dtype=torch.int64, device=A.device)
    st = lib().venom_prune(_ptr(A), A.stride(0) if R > 1 else max(K, A.stride(0)), R, K, V, N, M, _ptr(mask), K,
                           _ptr(kept), _ptr(total), _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_prune")
    return mask, kept, total


def venom_energy(kept_mass, total_mass, stream=None) -> float:
    """The energy metric from the per-block-row masses venom_prune returns."""
    e = ctypes.c_double(0.0)
    st = lib().venom_energy(_ptr(kept_mass), _ptr(total_mass), kept_mass.numel(), byref(e), _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_energy")
    return e.value


def venom_probe_smfmac_rate(iterations, sink, stream=None):
    """Launches the register-only matrix-instruction loop (the caller times it)."""
    st = lib().venom_probe_smfmac_rate(iterations, _ptr(sink), _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_probe_smfmac_rate")


def venom_import(values, columns, meta, R, K, V, N, M, stream=None) -> Handle:
    ws_owner, ws, nbytes = _workspace(R, K, V, N, M, values.device)
    out = c_void_p(0)
    st = lib().venom_import(_ptr(values), _ptr(columns), _ptr(meta), R, K, V, N, M, _ptr(ws), nbytes,
                            _stream_ptr(stream), byref(out))
    if st != VENOM_OK:
        raise VenomError(st, "venom_import")
    h = Handle(out, ws, R, K, V, N, M)
    h._owner = ws_owner
    return h


def venom_export(h: Handle, stream=None):
    """Returns (values int16 [R,G,2], columns int16 [R/V,G,4], meta int32 [R,ceil(G/8)]) CUDA tensors
    holding the canonical uint16 / uint32 bit patterns."""
    G = h.G
    dev = h.workspace.device
    values = torch.empty((h.R, G, 2), dtype=torch.int16, device=dev)
    columns = torch.empty((h.R // h.V, G, 4), dtype=torch.int16, device=dev)
    meta = torch.empty((h.R, (G + 7) // 8), dtype=torch.int32, device=dev)
    st = lib().venom_export(h.ptr, _ptr(values), _ptr(columns), _ptr(meta), _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_export")
    return values, columns, meta


def venom_decompress(h: Handle, out=None, stream=None):
    if out is None:
        out = torch.empty((h.R, h.K), dtype=torch.float16, device=h.workspace.device)
    st = lib().venom_decompress(h.ptr, _ptr(out), out.stride(0) if h.R > 1 else max(h.K, out.stride(0)),
                                _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_decompress")
    return out


ACTIVATIONS = {"none": 0, "gelu": 1, "gelu_tanh": 2}
_OUT_DTYPES = {torch.float16: 0, torch.float32: 1}


def _scratch_bytes(h: Handle, tokens) -> int:
    """Room for X transposed, its rows padded to whole 16-byte pieces (venom_linear_scratch_bytes, which the library
    checks the scratch against)."""
    return h.K * ((tokens + 7) // 8 * 8) * 2


def _new_scratch(nbytes, device, stream):
    """Scratch of a call on `stream` (None: the current one), from that stream's share of the caching allocator: dropped
    while the call's kernels are still to run, it is handed out again only to work that follows them on the stream."""
    if stream is None:
        return torch.empty(nbytes, dtype=torch.uint8, device=device)
    with torch.cuda.stream(stream):
        return torch.empty(nbytes, dtype=torch.uint8, device=device)


def _capturing(stream) -> bool:
    if stream is None:
        return _is_current_stream_capturing()
    with torch.cuda.stream(stream):
        return _is_current_stream_capturing()


class _KeptScratch:
    """The scratch buffers of one layer, one for each stream and thread that calls it (calls on different streams overlap, and
    two threads on one stream may queue their kernels between each other's), at most LIMIT of them, the oldest dropped
    first.  A call that is being captured gets one of its own from the graph's memory: the graph keeps using it."""

    LIMIT = 8

    def __init__(self):
        self._buffers = {}
        self._lock = threading.Lock()

    def get(self, nbytes, x, stream, stream_ptr):
        """(tensor, its address, its bytes), at least nbytes of them."""
        key = (stream_ptr, x.get_device(), get_ident())
        kept = self._buffers.get(key)
        capturing = _capturing(stream)
        if kept is not None and kept[2] >= nbytes and not capturing:
            return kept
        buf = _new_scratch(nbytes, x.device, stream)
        kept = (buf, buf.data_ptr(), buf.numel())
        if not capturing:
            with self._lock:
                self._buffers.pop(key, None)
                self._buffers[key] = kept
                while len(self._buffers) > self.LIMIT:
                    self._buffers.pop(next(iter(self._buffers)))
        return kept


def venom_spmm(h: Handle, B, out=None, out_dtype=None, variant=-1, stream=None, bias=None, activation="none"):
    """C = act(A . B + bias[:, None]).  B: K x C float16 CUDA tensor (unit column stride);
    bias: float16 CUDA vector of R entries or None; returns/fills C (R x C)."""
    assert B.is_cuda and B.dtype == torch.float16 and B.dim() == 2
    (rows, Ccols), (ldb, unit) = B.shape, B.stride()
    assert unit == 1
    if out is None:
        out = torch.empty((h.R, Ccols), dtype=out_dtype or torch.float16, device=B.device)
    dtype, strides = out.dtype, out.stride()
    assert dtype in _OUT_DTYPES and strides[1] == 1
    ldc = strides[0]
    if rows <= 1:
        ldb = max(Ccols, ldb)
    if out.shape[0] <= 1:
        ldc = max(Ccols, ldc)
    if bias is not None:
        assert bias.is_cuda and bias.dtype == torch.float16 and bias.dim() == 1 and bias.shape[0] == h.R
        assert bias.stride(0) == 1
    st = lib().venom_spmm_bias_act(h.ptr, B.data_ptr(), ldb, Ccols, _ptr(bias), ACTIVATIONS[activation], out.data_ptr(), ldc,
                                   _OUT_DTYPES[dtype], variant, _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_spmm")
    return out


def venom_linear(h: Handle, X, bias=None, activation="none", out=None, out_dtype=None, scratch=None, stream=None):
    """Y = act(X . A^T + bias): X tokens x K float16 CUDA tensor, Y tokens x R (token-major in and out).
    `scratch` (uint8 CUDA tensor) receives X transposed; allocated here when not given."""
    if scratch is None:
        assert X.is_cuda and X.dim() == 2
        scratch = _new_scratch(max(_scratch_bytes(h, X.shape[0]), 16), X.device, stream)
    return _linear(h, X, bias, activation, out, out_dtype, scratch.data_ptr(), scratch.numel(), _stream_ptr(stream))


def _linear(h, X, bias, activation, out, out_dtype, scratch_ptr, scratch_bytes, stream_ptr):
    assert X.is_cuda and X.dtype == torch.float16 and X.dim() == 2
    (tokens, K), (ldx, unit) = X.shape, X.stride()
    assert unit == 1 and K == h.K
    if out is None:
        out = torch.empty((tokens, h.R), dtype=out_dtype or torch.float16, device=X.device)
    dtype, (ldy, unit) = out.dtype, out.stride()
    assert dtype in _OUT_DTYPES and unit == 1 and out.shape == (tokens, h.R)
    if bias is not None:
        assert bias.is_cuda and bias.dtype == torch.float16 and bias.dim() == 1 and bias.shape[0] == h.R
    if tokens <= 1:
        ldx, ldy = max(h.K, ldx), max(h.R, ldy)
    st = lib().venom_linear(h.ptr, X.data_ptr(), ldx, tokens, _ptr(bias), ACTIVATIONS[activation], out.data_ptr(), ldy,
                            _OUT_DTYPES[dtype], scratch_ptr, scratch_bytes, stream_ptr)
    if st != VENOM_OK:
        raise VenomError(st, "venom_linear")
    return out


def venom_linear_static_max_bytes() -> int:
    return lib().venom_linear_static_max_bytes()


def venom_linear_static(h: Handle, X, out, bias=None, activation="none", stream=None):
    """venom_linear with the library's own static scratch: the caller passes the input and the output,
    nothing is allocated here or in the library."""
    assert X.is_cuda and X.dtype == torch.float16 and X.dim() == 2 and X.stride(1) == 1 and X.shape[1] == h.K
    tokens = X.shape[0]
    assert out.dtype in (torch.float16, torch.float32) and out.stride(1) == 1 and out.shape == (tokens, h.R)
    ldx = X.stride(0) if tokens > 1 else max(h.K, X.stride(0))
    ldy = out.stride(0) if tokens > 1 else max(h.R, out.stride(0))
    st = lib().venom_linear_static(h.ptr, _ptr(X), ldx, tokens, _ptr(bias), ACTIVATIONS[activation], _ptr(out), ldy,
                                   1 if out.dtype == torch.float32 else 0, _stream_ptr(stream))
    if st != VENOM_OK:
        raise VenomError(st, "venom_linear_static")
    return out


class Spmm:
    """The layer object of the paper's end-to-end section (its module listing): built once from a
    dense weight, a mask and a bias, it holds the compressed handle and is called like the linear
    layer it replaces, `y = layer(x)` with x tokens x K and y tokens x R.  Holds state only; every
    call is one venom_linear (the scratch for the transposed activations is kept between calls, one for each
    stream and thread that calls)."""

    def __init__(self, weight, mask, bias=None, V=128, N=2, M=8, activation="none"):
        self.handle = venom_compress(weight, mask, V, N, M)
        self.bias = bias
        self.activation = activation
        self._scratch = _KeptScratch()

    @classmethod
    def from_dense(cls, weight, bias=None, V=128, N=2, M=8, activation="none"):
        """Magnitude-prunes `weight` to V:N:M on the GPU (venom_prune), then compresses it."""
        mask, _, _ = venom_prune(weight, V, N, M)
        return cls(weight, mask, bias, V, N, M, activation)

    def __call__(self, x, out=None, out_dtype=None, stream=None):
        ptr = _stream_ptr(stream)
        h = self.handle
        scratch = self._scratch.get(max(_scratch_bytes(h, x.shape[0]), 16), x, stream, ptr)   # held until the call is queued
        return _linear(h, x, self.bias, self.activation, out, out_dtype, scratch[1], scratch[2], ptr)


def venom_get_info(h: Handle):
    R, K = c_int64(), c_int64()
    V, N, M = c_int(), c_int(), c_int()
    st = lib().venom_get_info(h.ptr, byref(R), byref(K), byref(V), byref(N), byref(M))
    if st != VENOM_OK:
        raise VenomError(st, "venom_get_info")
    return R.value, K.value, V.value, N.value, M.value


def venom_spmm_variants():
    L = lib()
    return [L.venom_spmm_variant_name(i).decode() for i in range(L.venom_spmm_variant_count())]


def venom_status_string(status: int) -> str:
    return lib().venom_status_string(status).decode()
