"""Python binding of libdpghost: argument marshalling only.

Each function has the name of the C entry point it calls and forwards torch
device tensors as raw pointers plus their row strides; every step of the
computation runs in the HIP kernels of libdpghost.so. Workspaces come from
torch's caching allocator; kernels run on torch's current stream unless a
stream is passed. Errors from the library raise DPError. There is no
fallback: if the library is not built, loading it raises.
"""
from __future__ import annotations

import contextlib
import ctypes
import os
from typing import Optional, Sequence

import torch

__all__ = [
    "DPError", "DP_F32", "DP_BF16", "DP_NORM_AUTO", "DP_NORM_GRAM", "DP_NORM_DIRECT",
    "lib", "library_path", "dp_abi_version",
    "dp_ghost_norm_linear", "dp_ghost_norm_linear_grouped", "dp_ghost_norm_embedding",
    "dp_tied_cross_term", "dp_clip_factors", "dp_clip_factors_scaled", "dp_clipped_grad_sum",
    "dp_embedding_rows", "dp_embedding_rows_add", "EmbeddingRows",
    "dp_clipped_grad_sum_grouped", "dp_clipped_grad_sum_noised_grouped", "dp_add_noise",
    "dp_grad_store_bytes", "dp_ghost_norm_linear_store", "dp_clipped_grad_sum_noised_store",
    "dp_noise_fill", "dp_vector_grads_grouped", "dp_vector_clipped_sum_noised_grouped",
    "dp_ghost_norm_linear_bias_grouped", "VectorSums",
    "dp_ghost_norm_positional", "dp_clipped_grad_sum_positional_noised",
    "LinearGroup", "VectorGroup",
]

DP_F32, DP_BF16 = 0, 1
DP_NORM_AUTO, DP_NORM_GRAM, DP_NORM_DIRECT = 0, 1, 2

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB: Optional[ctypes.CDLL] = None


class DPError(RuntimeError):
    pass


class dp_linear_t(ctypes.Structure):
    _fields_ = [("A", ctypes.c_void_p), ("lda", ctypes.c_int64), ("d_in", ctypes.c_int32),
                ("G", ctypes.c_void_p), ("ldg", ctypes.c_int64), ("d_out", ctypes.c_int32),
                ("algo", ctypes.c_int32)]


class dp_vector_t(ctypes.Structure):
    _fields_ = [("X", ctypes.c_void_p), ("ldx", ctypes.c_int64), ("G", ctypes.c_void_p),
                ("ldg", ctypes.c_int64), ("d", ctypes.c_int32)]


def library_path() -> str:
    """libdpghost.so beside this file, or the library that DPGHOST_LIBRARY
    names (a build of the host code with sanitizers, say)."""
    return os.environ.get("DPGHOST_LIBRARY") or os.path.join(_HERE, "libdpghost.so")


_VP, _I, _I64, _U64, _F, _SZ = (ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_uint64,
                                ctypes.c_float, ctypes.c_size_t)
_SIGS = {
    "dp_abi_version": ([], _I),
    "dp_status_string": ([_I], ctypes.c_char_p),
    "dp_last_error": ([], ctypes.c_char_p),
    "dp_ghost_norm_linear_workspace": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I], _SZ),
    "dp_ghost_norm_linear_bias_workspace": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP), _I,
                                             _I, _I, _I], _SZ),
    "dp_ghost_norm_linear_bias_grouped": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP), _I,
                                           _I, _I, _I, _VP, _I, _VP, _SZ, _VP], _I),
    "dp_ghost_norm_linear_bias_grouped_noalloc": ([ctypes.POINTER(dp_linear_t),
                                                   ctypes.POINTER(_VP), _I, _I, _I, _I, _VP, _I,
                                                   _VP], _I),
    "dp_ghost_norm_linear_grouped": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I, _VP, _I,
                                      _VP, _SZ, _VP], _I),
    "dp_ghost_norm_linear": ([_VP, _I64, _VP, _I64, _I, _I, _I, _I, _I, _I, _VP, _I, _VP, _SZ,
                              _VP], _I),
    "dp_ghost_norm_embedding_workspace": ([_I, _I, _I], _SZ),
    "dp_ghost_norm_embedding": ([_VP, _VP, _I64, _I, _I, _I, _I, _I, _VP, _I, _VP, _VP, _VP,
                                 _SZ, _VP], _I),
    "dp_tied_cross_term_workspace": ([_I, _I, _I], _SZ),
    "dp_tied_cross_term": ([_VP, _VP, _I64, _VP, _I64, _VP, _I64, _I, _I, _I, _I, _I, _F, _VP,
                            _I, _VP, _SZ, _VP], _I),
    "dp_clip_factors": ([_VP, _I, _F, _VP, _VP], _I),
    "dp_clipped_grad_sum_workspace": ([_I, _I, _I, _I], _SZ),
    "dp_embedding_rows_workspace": ([_I, _I, _I], _SZ),
    "dp_embedding_rows": ([_VP, _I64, _VP, _VP, _I, _I, _I, _I, _I, _VP, _SZ, _VP], _I),
    "dp_embedding_rows_add": ([_VP, _SZ, _I, _I, _I, _I, _I, _VP, _VP], _I),
    "dp_clipped_grad_sum": ([_VP, _I64, _VP, _I64, _VP, _VP, _I, _I, _I, _I, _I, _I, _VP, _I,
                             _VP, _SZ, _VP], _I),
    "dp_clipped_grad_sum_grouped": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP), _I, _VP,
                                     _I, _I, _I, _I, _I, _VP], _I),
    "dp_clipped_grad_sum_grouped_ws": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP), _I, _VP,
                                        _I, _I, _I, _I, _I, _VP, _SZ, _VP], _I),
    "dp_clipped_grad_sum_noised_grouped": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP),
                                            ctypes.POINTER(_U64), ctypes.POINTER(ctypes.c_int32),
                                            _I, _VP, _I, _I, _I, _I, _F, _F, _I, _U64, _U64, _VP],
                                           _I),
    "dp_add_noise": ([_VP, _I64, _F, _F, _I, _U64, _U64, _U64, _VP], _I),
    "dp_clipped_grad_sum_noised_grouped_workspace": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I,
                                                      _I], _SZ),
    "dp_clipped_grad_sum_split_workspace": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I, _I],
                                            _SZ),
    "dp_clipped_grad_sum_noised_grouped_ws": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP),
                                               ctypes.POINTER(_U64), ctypes.POINTER(ctypes.c_int32),
                                               _I, _VP, _I, _I, _I, _I, _F, _F, _I, _U64, _U64,
                                               _VP, _SZ, _VP], _I),
    "dp_grad_store_bytes": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I], _SZ),
    "dp_ghost_norm_linear_store": ([ctypes.POINTER(dp_linear_t), _I, _I, _I, _I, _VP, _I, _VP,
                                    _SZ, _VP], _I),
    "dp_clipped_grad_sum_noised_store": ([ctypes.POINTER(dp_linear_t), ctypes.POINTER(_VP),
                                          ctypes.POINTER(_U64), ctypes.POINTER(ctypes.c_int32),
                                          ctypes.POINTER(ctypes.c_int32), _I, _VP, _I, _I, _I,
                                          _F, _F, _I, _U64, _U64, _VP, _SZ, _VP], _I),
    "dp_clip_factors_scaled": ([_VP, _I, _F, _F, _VP, _VP, _VP], _I),
    "dp_clip_factors_scaled2": ([_VP, _VP, _I, _F, _F, _VP, _VP, _VP], _I),
    "dp_noise_fill": ([_VP, _I64, _F, _F, _I, _U64, _U64, _U64, _VP], _I),
    "dp_vector_grads_workspace": ([ctypes.POINTER(dp_vector_t), _I, _I, _I, _I], _SZ),
    "dp_vector_grads_grouped": ([ctypes.POINTER(dp_vector_t), _I, _I, _I, _I,
                                 ctypes.POINTER(_VP), _VP, _I, _VP, _SZ, _VP], _I),
    "dp_vector_clipped_sum_noised_grouped": ([ctypes.POINTER(_VP), ctypes.POINTER(ctypes.c_int32),
                                              _I, _I, _VP, ctypes.POINTER(_VP),
                                              ctypes.POINTER(_U64), ctypes.POINTER(ctypes.c_int32),
                                              _F, _F, _I, _U64, _U64, _VP], _I),
    "dp_ghost_norm_positional_workspace": ([_I, _I, _I], _SZ),
    "dp_ghost_norm_positional": ([_VP, _I64, _I, _I, _I, _I, _VP, _I, _VP, _SZ, _VP], _I),
    "dp_clipped_grad_sum_positional_noised": ([_VP, _I64, _VP, _I, _I, _I, _I, _VP, _I, _I64,
                                               _U64, _I, _F, _F, _I, _U64, _U64, _VP], _I),
}


def lib() -> ctypes.CDLL:
    """Loads libdpghost.so from the package directory (it must be built)."""
    global _LIB
    if _LIB is None:
        path = library_path()
        if not os.path.exists(path):
            raise DPError(f"{path} is not built; run `python -m paper_2609_40335_amd.build`")
        L = ctypes.CDLL(path)
        for name, (args, res) in _SIGS.items():
            f = getattr(L, name)
            f.argtypes = args
            f.restype = res
        _LIB = L
    return _LIB


def _check(status: int, name: str) -> None:
    if status != 0:
        L = lib()
        raise DPError(f"{name}: {L.dp_status_string(status).decode()}: "
                      f"{L.dp_last_error().decode()}")


def _dtype(t: torch.Tensor) -> int:
    if t.dtype == torch.bfloat16:
        return DP_BF16
    if t.dtype == torch.float32:
        return DP_F32
    raise DPError(f"unsupported dtype {t.dtype}")


def _rows(t: torch.Tensor, name: str):
    """(pointer, B, T, width, row stride) of a token-major [B, T, w] tensor."""
    if t.dim() != 3:
        raise DPError(f"{name} must be [B, T, w]")
    B, T, w = t.shape
    if t.stride(2) != 1 or (B > 1 and t.stride(0) != T * t.stride(1)):
        raise DPError(f"{name} must have unit feature stride and uniformly spaced token rows")
    return t.data_ptr(), B, T, w, t.stride(1)


def _dev(t: torch.Tensor, name: str) -> None:
    if not t.is_cuda:
        raise DPError(f"{name} must be a device tensor")


def _stream(stream) -> int:
    s = torch.cuda.current_stream() if stream is None else stream
    return s.cuda_stream


def _on(stream):
    """Context whose allocations come from ``stream``'s own pool. A call's scratch must:
    the current stream's pool hands out memory that kernels queued there may still use,
    which only calls on that same stream wait for."""
    if stream is None:
        return contextlib.nullcontext()
    if not isinstance(stream, torch.cuda.Stream):
        stream = torch.cuda.ExternalStream(stream.cuda_stream)
    return torch.cuda.stream(stream)


def _ws(nbytes: int, device, stream=None) -> torch.Tensor:
    """Scratch of a call on ``stream`` (None: the current one)."""
    if stream is None:
        return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device=device)
    with _on(stream):
        return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device=device)


def _split_bytes(descs, n: int, B: int, T: int, dt: int, transpose_out) -> int:
    """Workspace bytes of a clipped sum's split tail (0: nothing is split)."""
    return lib().dp_clipped_grad_sum_split_workspace(descs, n, B, T, dt, int(transpose_out))


def dp_abi_version() -> int:
    return lib().dp_abi_version()


def _layer(A, G, algo=DP_NORM_AUTO) -> dp_linear_t:
    _dev(A, "A"); _dev(G, "G")
    pa, B, T, d_in, lda = _rows(A, "A")
    pg, B2, T2, d_out, ldg = _rows(G, "G")
    if (B, T) != (B2, T2):
        raise DPError("A and G must share B and T")
    if A.dtype != G.dtype:
        raise DPError("A and G must share a dtype")
    return dp_linear_t(pa, lda, d_in, pg, ldg, d_out, algo)


def dp_ghost_norm_linear_bias_grouped(layers: Sequence, bias_grads: Sequence, norm2: torch.Tensor,
                                      accumulate: bool = False, stream=None) -> torch.Tensor:
    """The grouped norm that also writes bias_grads[l] (fp32 [B, d_out], or
    None for a layer without bias) = sum over tokens of G_l, norms included."""
    with _on(stream):  # the group and its workspace live for this call only
        group = LinearGroup(layers, bias_grads=bias_grads)
    return group.ghost_norm(norm2, accumulate, stream)


def dp_ghost_norm_linear_bias_grouped_noalloc(layers: Sequence, bias_grads: Optional[Sequence],
                                              norm2: torch.Tensor, accumulate: bool = False,
                                              stream=None) -> torch.Tensor:
    """The grouped norm (with optional bias gradients) in the library's static
    device scratch: no workspace is allocated here or in the library."""
    descs = [_layer(*l) for l in layers]
    A0 = layers[0][0]
    B, T = A0.shape[0], A0.shape[1]
    for l in layers:
        if tuple(l[0].shape[:2]) != (B, T) or l[0].dtype != A0.dtype:
            raise DPError("all layers of a group share B, T and dtype")
    arr = (dp_linear_t * len(descs))(*descs)
    bias = None
    if bias_grads is not None:
        if len(bias_grads) != len(descs):
            raise DPError("one bias gradient (or None) per layer")
        for l, g in zip(layers, bias_grads):
            if g is not None and (g.dtype != torch.float32 or not g.is_contiguous()
                                  or tuple(g.shape) != (B, l[1].shape[2])):
                raise DPError("bias gradients must be contiguous fp32 [B, d_out]")
        bias = (ctypes.c_void_p * len(descs))(*[None if g is None else g.data_ptr()
                                                for g in bias_grads])
    _check(lib().dp_ghost_norm_linear_bias_grouped_noalloc(arr, bias, len(descs), B, T,
                                                          _dtype(A0), norm2.data_ptr(),
                                                          int(accumulate), _stream(stream)),
           "dp_ghost_norm_linear_bias_grouped_noalloc")
    return norm2


def dp_ghost_norm_linear_grouped(layers: Sequence, norm2: torch.Tensor, accumulate: bool = False,
                                 stream=None) -> torch.Tensor:
    """layers: sequence of (A, G) or (A, G, algo); norm2: fp32 [B]."""
    L = lib()
    descs = [_layer(*l) for l in layers]
    A0 = layers[0][0]
    B, T = A0.shape[0], A0.shape[1]
    for l in layers:
        if tuple(l[0].shape[:2]) != (B, T) or l[0].dtype != A0.dtype:
            raise DPError("all layers of a group share B, T and dtype")
    arr = (dp_linear_t * len(descs))(*descs)
    dt = _dtype(A0)
    nbytes = L.dp_ghost_norm_linear_workspace(arr, len(descs), B, T, dt)
    ws = _ws(nbytes, A0.device, stream)
    _check(L.dp_ghost_norm_linear_grouped(arr, len(descs), B, T, dt, norm2.data_ptr(),
                                          int(accumulate), ws.data_ptr(), ws.numel(),
                                          _stream(stream)), "dp_ghost_norm_linear_grouped")
    return norm2


def dp_ghost_norm_linear(A, G, norm2, accumulate: bool = False, algo: int = DP_NORM_AUTO,
                         stream=None) -> torch.Tensor:
    L = lib()
    d = _layer(A, G, algo)
    B, T = A.shape[0], A.shape[1]
    dt = _dtype(A)
    nbytes = L.dp_ghost_norm_linear_workspace(ctypes.byref(d), 1, B, T, dt)
    ws = _ws(nbytes, A.device, stream)
    _check(L.dp_ghost_norm_linear(d.A, d.lda, d.G, d.ldg, B, T, d.d_in, d.d_out, dt, algo,
                                  norm2.data_ptr(), int(accumulate), ws.data_ptr(), ws.numel(),
                                  _stream(stream)), "dp_ghost_norm_linear")
    return norm2


def dp_ghost_norm_embedding(ids, dE, V: int, norm2, accumulate: bool = False, seg_id=None,
                            n_unique=None, stream=None) -> torch.Tensor:
    L = lib()
    _dev(ids, "ids"); _dev(dE, "dE")
    pe, B, T, d, lde = _rows(dE, "dE")
    if ids.dtype != torch.int32 or tuple(ids.shape) != (B, T) or not ids.is_contiguous():
        raise DPError("ids must be contiguous int32 [B, T]")
    ws = _ws(L.dp_ghost_norm_embedding_workspace(B, T, d), dE.device, stream)
    _check(L.dp_ghost_norm_embedding(ids.data_ptr(), pe, lde, B, T, V, d, _dtype(dE),
                                     norm2.data_ptr(), int(accumulate),
                                     None if seg_id is None else seg_id.data_ptr(),
                                     None if n_unique is None else n_unique.data_ptr(),
                                     ws.data_ptr(), ws.numel(), _stream(stream)),
           "dp_ghost_norm_embedding")
    return norm2


def dp_tied_cross_term(ids, dE, H, Gz, V: int, out, scale: float = 1.0,
                       accumulate: bool = False, stream=None) -> torch.Tensor:
    """Gz: [B, T, V] (may be a column slice of a row-padded tensor)."""
    L = lib()
    for t, n in ((ids, "ids"), (dE, "dE"), (H, "H"), (Gz, "Gz")):
        _dev(t, n)
    pe, B, T, d, lde = _rows(dE, "dE")
    ph, _, _, _, ldh = _rows(H, "H")
    pz, _, _, Vz, ldz = _rows(Gz, "Gz")
    if Vz < V:
        raise DPError("Gz must have at least V columns")
    if ids.dtype != torch.int32 or tuple(ids.shape) != (B, T) or not ids.is_contiguous():
        raise DPError("ids must be contiguous int32 [B, T]")
    ws = _ws(L.dp_tied_cross_term_workspace(B, T, d), dE.device, stream)
    _check(L.dp_tied_cross_term(ids.data_ptr(), pe, lde, ph, ldh, pz, ldz, B, T, V, d,
                                _dtype(dE), float(scale), out.data_ptr(), int(accumulate),
                                ws.data_ptr(), ws.numel(), _stream(stream)),
           "dp_tied_cross_term")
    return out


def dp_clip_factors(norm2, C: float, c, stream=None) -> torch.Tensor:
    _check(lib().dp_clip_factors(norm2.data_ptr(), norm2.numel(), float(C), c.data_ptr(),
                                 _stream(stream)), "dp_clip_factors")
    return c


def dp_clip_factors_scaled(norm2, C: float, scale: float, c_scaled, c=None,
                           stream=None) -> torch.Tensor:
    """c_scaled = scale * clip factors (and the factors into c when given)."""
    _check(lib().dp_clip_factors_scaled(norm2.data_ptr(), norm2.numel(), float(C), float(scale),
                                        None if c is None else c.data_ptr(),
                                        c_scaled.data_ptr(), _stream(stream)),
           "dp_clip_factors_scaled")
    return c_scaled


def dp_clip_factors_scaled2(norm2_a, norm2_b, C: float, scale: float, c_scaled, c=None,
                            stream=None) -> torch.Tensor:
    """dp_clip_factors_scaled of norm2_a + norm2_b."""
    _check(lib().dp_clip_factors_scaled2(norm2_a.data_ptr(), norm2_b.data_ptr(), norm2_a.numel(),
                                         float(C), float(scale), None if c is None else c.data_ptr(),
                                         c_scaled.data_ptr(), _stream(stream)),
           "dp_clip_factors_scaled2")
    return c_scaled


def dp_clipped_grad_sum(A, G, c, out, ids=None, V: Optional[int] = None,
                        transpose_out: bool = False, accumulate: bool = False,
                        stream=None) -> torch.Tensor:
    """Linear form: A [B,T,d_in], G [B,T,d_out]; embedding form: A None, ids [B,T], V."""
    L = lib()
    _dev(G, "G")
    pg, B, T, d_out, ldg = _rows(G, "G")
    dt = _dtype(G)
    if ids is None:
        _dev(A, "A")
        pa, _, _, d_in, lda = _rows(A, "A")
        desc = (dp_linear_t * 1)(dp_linear_t(pa, lda, d_in, pg, ldg, d_out, DP_NORM_AUTO))
        nbytes = _split_bytes(desc, 1, B, T, dt, transpose_out)
        ws = _ws(nbytes, G.device, stream) if nbytes else None
        outs = (ctypes.c_void_p * 1)(out.data_ptr())
        _check(L.dp_clipped_grad_sum_grouped_ws(desc, outs, 1, c.data_ptr(), B, T, dt,
                                                int(transpose_out), int(accumulate),
                                                None if ws is None else ws.data_ptr(),
                                                0 if ws is None else ws.numel(),
                                                _stream(stream)),
               "dp_clipped_grad_sum")
        return out
    if A is not None or V is None:
        raise DPError("embedding form takes ids and V, not A")
    if ids.dtype != torch.int32 or tuple(ids.shape) != (B, T) or not ids.is_contiguous():
        raise DPError("ids must be contiguous int32 [B, T]")
    ws = _ws(L.dp_clipped_grad_sum_workspace(B, T, d_out, 1), G.device, stream)
    _check(L.dp_clipped_grad_sum(None, 0, pg, ldg, ids.data_ptr(), c.data_ptr(), B, T, V, d_out,
                                 dt, int(transpose_out), out.data_ptr(), int(accumulate),
                                 ws.data_ptr(), ws.numel(), _stream(stream)),
           "dp_clipped_grad_sum")
    return out


class EmbeddingRows:
    """The embedding form of the clipped sum in two calls on one workspace:
    compute() writes one row per distinct id (c-weighted sums of G's rows)
    and touches nothing else; add_to() adds those rows onto the [V, d] (or
    transposed) output, bit for bit as dp_clipped_grad_sum(..., ids=ids,
    accumulate=True) would. add_to() must be ordered after compute()."""

    def __init__(self, B: int, T: int, V: int, d: int, device=None):
        self.B, self.T, self.V, self.d = B, T, V, d
        L = lib()
        n = L.dp_embedding_rows_workspace(B, T, d)
        if n == 0:
            raise DPError("B, T and d must be positive")
        self.ws = _ws(n, device if device is not None else torch.device("cuda"))

    def compute(self, G, ids, c, stream=None) -> None:
        dp_embedding_rows(G, ids, c, self.V, self.ws, stream=stream)

    def add_to(self, out, transpose_out: bool = False, stream=None) -> None:
        dp_embedding_rows_add(self.ws, self.B, self.T, self.V, self.d, out,
                              transpose_out=transpose_out, stream=stream)


def dp_embedding_rows(G, ids, c, V: int, ws, stream=None) -> None:
    L = lib()
    _dev(G, "G")
    pg, B, T, d, ldg = _rows(G, "G")
    if ids.dtype != torch.int32 or tuple(ids.shape) != (B, T) or not ids.is_contiguous():
        raise DPError("ids must be contiguous int32 [B, T]")
    _check(L.dp_embedding_rows(pg, ldg, ids.data_ptr(), c.data_ptr(), B, T, V, d, _dtype(G),
                               ws.data_ptr(), ws.numel() * ws.element_size(), _stream(stream)),
           "dp_embedding_rows")


def dp_embedding_rows_add(ws, B: int, T: int, V: int, d: int, out, transpose_out: bool = False,
                          stream=None) -> None:
    L = lib()
    if out.dtype != torch.float32 or not out.is_contiguous():
        raise DPError("out must be contiguous float32")
    if tuple(out.shape) != ((d, V) if transpose_out else (V, d)):
        raise DPError("out must be [V, d] ([d, V] with transpose_out)")
    _check(L.dp_embedding_rows_add(ws.data_ptr(), ws.numel() * ws.element_size(), B, T, V, d,
                                   int(transpose_out), out.data_ptr(), _stream(stream)),
           "dp_embedding_rows_add")


def dp_clipped_grad_sum_grouped(layers: Sequence, outs: Sequence[torch.Tensor], c,
                                transpose_out: bool = False, accumulate: bool = False,
                                stream=None) -> None:
    L = lib()
    descs = [_layer(l[0], l[1]) for l in layers]
    arr = (dp_linear_t * len(descs))(*descs)
    optrs = (ctypes.c_void_p * len(outs))(*[o.data_ptr() for o in outs])
    A0 = layers[0][0]
    _check(L.dp_clipped_grad_sum_grouped(arr, optrs, len(descs), c.data_ptr(), A0.shape[0],
                                         A0.shape[1], _dtype(A0), int(transpose_out),
                                         int(accumulate), _stream(stream)),
           "dp_clipped_grad_sum_grouped")


def _noise_arrays(n: int, tensor_ids: Sequence[int], accumulate):
    if len(tensor_ids) != n:
        raise DPError("one tensor id per layer")
    tids = (ctypes.c_uint64 * n)(*[int(t) for t in tensor_ids])
    if accumulate is None or isinstance(accumulate, (bool, int)):
        acc = (ctypes.c_int32 * n)(*([int(bool(accumulate))] * n))
    else:
        if len(accumulate) != n:
            raise DPError("one accumulate flag per layer")
        acc = (ctypes.c_int32 * n)(*[int(bool(a)) for a in accumulate])
    return tids, acc


def dp_clipped_grad_sum_noised_grouped(layers: Sequence, outs: Sequence[torch.Tensor], c,
                                       tensor_ids: Sequence[int], sigma: float, C: float,
                                       B_norm: int, seed: int, step: int, accumulate=None,
                                       transpose_out: bool = False, stream=None) -> None:
    """Clipped sums with the Gaussian mechanism fused into their store; the
    noise each output gets is the one dp_add_noise(outs[l], ..., tensor_ids[l],
    step) would add. ``accumulate`` is a bool or one bool per layer. (No
    workspace: the last round of tiles is not split; LinearGroup passes one.)"""
    L = lib()
    descs = [_layer(l[0], l[1]) for l in layers]
    arr = (dp_linear_t * len(descs))(*descs)
    optrs = (ctypes.c_void_p * len(outs))(*[o.data_ptr() for o in outs])
    tids, acc = _noise_arrays(len(descs), tensor_ids, accumulate)
    A0 = layers[0][0]
    _check(L.dp_clipped_grad_sum_noised_grouped(arr, optrs, tids, acc, len(descs), c.data_ptr(),
                                                A0.shape[0], A0.shape[1], _dtype(A0),
                                                int(transpose_out), float(sigma), float(C),
                                                int(B_norm), int(seed), int(step),
                                                _stream(stream)),
           "dp_clipped_grad_sum_noised_grouped")


def dp_add_noise(grad, sigma: float, C: float, B_norm: int, seed: int, tensor_id: int,
                 step: int, stream=None) -> torch.Tensor:
    if grad.dtype != torch.float32 or not grad.is_contiguous():
        raise DPError("grad must be contiguous fp32")
    _check(lib().dp_add_noise(grad.data_ptr(), grad.numel(), float(sigma), float(C), int(B_norm),
                              int(seed), int(tensor_id), int(step), _stream(stream)),
           "dp_add_noise")
    return grad


def dp_noise_fill(out, sigma: float, C: float, B_norm: int, seed: int, tensor_id: int,
                  step: int, stream=None) -> torch.Tensor:
    """out = sigma*C*z / B_norm: dp_add_noise on zeros, without reading out."""
    if out.dtype != torch.float32 or not out.is_contiguous():
        raise DPError("out must be contiguous fp32")
    _check(lib().dp_noise_fill(out.data_ptr(), out.numel(), float(sigma), float(C), int(B_norm),
                               int(seed), int(tensor_id), int(step), _stream(stream)),
           "dp_noise_fill")
    return out


def _vector(X, G) -> dp_vector_t:
    _dev(G, "G")
    pg, B, T, d, ldg = _rows(G, "G")
    if X is None:
        return dp_vector_t(None, 0, pg, ldg, d)
    _dev(X, "X")
    px, B2, T2, d2, ldx = _rows(X, "X")
    if (B, T, d) != (B2, T2, d2) or X.dtype != G.dtype:
        raise DPError("X and G must share shape and dtype")
    return dp_vector_t(px, ldx, pg, ldg, d)


def dp_vector_grads_grouped(params: Sequence, grads: Sequence[torch.Tensor], norm2=None,
                            accumulate: bool = False, stream=None) -> None:
    """params: (X or None, G) per vector parameter, [B, T, d] each; grads:
    fp32 [B, d] outputs (the per-example gradients); norm2 (optional) gets
    their squared norms added (accumulate) or written."""
    L = lib()
    descs = (dp_vector_t * len(params))(*[_vector(*p) for p in params])
    G0 = params[0][1]
    B, T, dt = G0.shape[0], G0.shape[1], _dtype(G0)
    for (X, G), g in zip(params, grads):
        if tuple(G.shape[:2]) != (B, T) or _dtype(G) != dt:
            raise DPError("all parameters of a group share B, T and dtype")
        if g.dtype != torch.float32 or tuple(g.shape) != (B, G.shape[2]) or not g.is_contiguous():
            raise DPError("grads must be contiguous fp32 [B, d]")
    if len(grads) != len(params):
        raise DPError("one gradient buffer per parameter")
    gp = (ctypes.c_void_p * len(grads))(*[g.data_ptr() for g in grads])
    ws = _ws(L.dp_vector_grads_workspace(descs, len(params), B, T, dt), G0.device, stream)
    _check(L.dp_vector_grads_grouped(descs, len(params), B, T, dt, gp,
                                     None if norm2 is None else norm2.data_ptr(), int(accumulate),
                                     ws.data_ptr(), ws.numel(), _stream(stream)),
           "dp_vector_grads_grouped")


def dp_vector_clipped_sum_noised_grouped(grads: Sequence[torch.Tensor], outs: Sequence[torch.Tensor],
                                         c, tensor_ids: Sequence[int], sigma: float, C: float,
                                         B_norm: int, seed: int, step: int, accumulate=None,
                                         stream=None) -> None:
    """outs[v] = (prior + sum_i c_i grads[v][i] + sigma C z) / B_norm."""
    n = len(grads)
    if len(outs) != n:
        raise DPError("one output per parameter")
    for g, o in zip(grads, outs):
        if o.dtype != torch.float32 or o.numel() != g.shape[1] or not o.is_contiguous():
            raise DPError("outs must be contiguous fp32 with d elements")
    gp = (ctypes.c_void_p * n)(*[g.data_ptr() for g in grads])
    op = (ctypes.c_void_p * n)(*[o.data_ptr() for o in outs])
    dd = (ctypes.c_int32 * n)(*[int(g.shape[1]) for g in grads])
    tids, acc = _noise_arrays(n, tensor_ids, accumulate)
    _check(lib().dp_vector_clipped_sum_noised_grouped(gp, dd, n, int(grads[0].shape[0]),
                                                      c.data_ptr(), op, tids, acc, float(sigma),
                                                      float(C), int(B_norm), int(seed), int(step),
                                                      _stream(stream)),
           "dp_vector_clipped_sum_noised_grouped")


class VectorSums:
    """Noised clipped sums of many vector parameters from per-example
    gradients already in memory (fp32 [B, d] each: from dp_vector_grads_grouped
    or from a fused bias), pointer arrays prepared once."""

    def __init__(self, grads: Sequence[torch.Tensor], outs: Sequence[torch.Tensor],
                 tensor_ids: Sequence[int], accumulate=None):
        n = len(grads)
        if n == 0 or len(outs) != n:
            raise DPError("one output per gradient, at least one")
        B = grads[0].shape[0]
        for g, o in zip(grads, outs):
            if g.dtype != torch.float32 or g.dim() != 2 or g.shape[0] != B or not g.is_contiguous():
                raise DPError("grads must be contiguous fp32 [B, d] with one B")
            if o.dtype != torch.float32 or o.numel() != g.shape[1] or not o.is_contiguous():
                raise DPError("outs must be contiguous fp32 with d elements")
        self._keep = (list(grads), list(outs))
        self.n, self.B = n, int(B)
        self._gp = (ctypes.c_void_p * n)(*[g.data_ptr() for g in grads])
        self._op = (ctypes.c_void_p * n)(*[o.data_ptr() for o in outs])
        self._dd = (ctypes.c_int32 * n)(*[int(g.shape[1]) for g in grads])
        self._tids, self._acc = _noise_arrays(n, tensor_ids, accumulate)

    def noised(self, c, sigma: float, C: float, B_norm: int, seed: int, step: int,
               stream=None) -> None:
        _check(lib().dp_vector_clipped_sum_noised_grouped(self._gp, self._dd, self.n, self.B,
                                                          c.data_ptr(), self._op, self._tids,
                                                          self._acc, float(sigma), float(C),
                                                          int(B_norm), int(seed), int(step),
                                                          _stream(stream)),
               "dp_vector_clipped_sum_noised_grouped")


def dp_ghost_norm_positional(dE, norm2, accumulate: bool = False, stream=None) -> torch.Tensor:
    """norm2[i] (+)= sum_t ||dE[i, t]||^2 (the position table's per-example norm)."""
    L = lib()
    _dev(dE, "dE")
    pe, B, T, d, lde = _rows(dE, "dE")
    ws = _ws(L.dp_ghost_norm_positional_workspace(B, T, d), dE.device, stream)
    _check(L.dp_ghost_norm_positional(pe, lde, B, T, d, _dtype(dE), norm2.data_ptr(),
                                      int(accumulate), ws.data_ptr(), ws.numel(), _stream(stream)),
           "dp_ghost_norm_positional")
    return norm2


def dp_clipped_grad_sum_positional_noised(dE, c, out, tensor_id: int, sigma: float, C: float,
                                          B_norm: int, seed: int, step: int,
                                          accumulate: bool = False, stream=None) -> torch.Tensor:
    """out [n_pos, d] fp32: rows t < T get sum_i c_i dE[i, t]; all rows the noise."""
    _dev(dE, "dE")
    pe, B, T, d, lde = _rows(dE, "dE")
    if out.dtype != torch.float32 or out.dim() != 2 or out.shape[1] != d or out.stride(1) != 1:
        raise DPError("out must be fp32 [n_pos, d] with unit column stride")
    _check(lib().dp_clipped_grad_sum_positional_noised(pe, lde, c.data_ptr(), B, T, d, _dtype(dE),
                                                       out.data_ptr(), out.shape[0], out.stride(0),
                                                       int(tensor_id), int(accumulate),
                                                       float(sigma), float(C), int(B_norm),
                                                       int(seed), int(step), _stream(stream)),
           "dp_clipped_grad_sum_positional_noised")
    return out


class VectorGroup:
    """Descriptors, per-example gradient buffers and workspace of many vector
    parameters of one batch, prepared once (see dp_vector_grads_grouped)."""

    def __init__(self, params: Sequence):
        L = lib()
        self._tensors = [t for p in params for t in p if t is not None]
        self.n = len(params)
        self.descs = (dp_vector_t * self.n)(*[_vector(*p) for p in params])
        G0 = params[0][1]
        self.B, self.T, self.dt = G0.shape[0], G0.shape[1], _dtype(G0)
        self.d = [int(p[1].shape[2]) for p in params]
        self.grads = [torch.empty(self.B, d, device=G0.device) for d in self.d]
        self._gp = (ctypes.c_void_p * self.n)(*[g.data_ptr() for g in self.grads])
        self._dd = (ctypes.c_int32 * self.n)(*self.d)
        self.ws = _ws(L.dp_vector_grads_workspace(self.descs, self.n, self.B, self.T, self.dt),
                      G0.device)
        self._noise_key = None

    def grads_and_norm(self, norm2, accumulate: bool = False, stream=None) -> None:
        _check(lib().dp_vector_grads_grouped(self.descs, self.n, self.B, self.T, self.dt, self._gp,
                                             None if norm2 is None else norm2.data_ptr(),
                                             int(accumulate), self.ws.data_ptr(), self.ws.numel(),
                                             _stream(stream)), "dp_vector_grads_grouped")

    def clipped_sum_noised(self, c, outs: Sequence[torch.Tensor], tensor_ids: Sequence[int],
                           sigma: float, C: float, B_norm: int, seed: int, step: int,
                           accumulate=None, stream=None) -> None:
        key = (tuple(o.data_ptr() for o in outs), tuple(int(t) for t in tensor_ids),
               accumulate if isinstance(accumulate, (bool, int, type(None)))
               else tuple(bool(a) for a in accumulate))
        if self._noise_key != key:
            self._noise_key = key
            self._op = (ctypes.c_void_p * self.n)(*[o.data_ptr() for o in outs])
            self._na = _noise_arrays(self.n, tensor_ids, accumulate)
        tids, acc = self._na
        _check(lib().dp_vector_clipped_sum_noised_grouped(self._gp, self._dd, self.n, self.B,
                                                          c.data_ptr(), self._op, tids, acc,
                                                          float(sigma), float(C), int(B_norm),
                                                          int(seed), int(step), _stream(stream)),
               "dp_vector_clipped_sum_noised_grouped")


def dp_grad_store_bytes(layers: Sequence) -> int:
    """Bytes of the per-example gradient store for these (A, G) layers; 0 when
    the store form does not apply (bf16, T % 32 == 0, 16-byte rows)."""
    descs = [_layer(l[0], l[1]) for l in layers]
    arr = (dp_linear_t * len(descs))(*descs)
    A0 = layers[0][0]
    return lib().dp_grad_store_bytes(arr, len(descs), A0.shape[0], A0.shape[1], _dtype(A0))


def dp_ghost_norm_linear_store(layers: Sequence, norm2: torch.Tensor, store: torch.Tensor,
                               accumulate: bool = False, stream=None) -> torch.Tensor:
    """Direct norms of every layer, each example's gradient tiles kept in
    ``store`` (a byte tensor of dp_grad_store_bytes(layers) bytes)."""
    descs = [_layer(l[0], l[1]) for l in layers]
    arr = (dp_linear_t * len(descs))(*descs)
    A0 = layers[0][0]
    _check(lib().dp_ghost_norm_linear_store(arr, len(descs), A0.shape[0], A0.shape[1],
                                            _dtype(A0), norm2.data_ptr(), int(accumulate),
                                            store.data_ptr(), store.numel() * store.element_size(),
                                            _stream(stream)),
           "dp_ghost_norm_linear_store")
    return norm2


def _flags(n: int, flags, what: str):
    """A bool for every layer, or one bool per layer, as a ctypes int32 array."""
    if flags is None or isinstance(flags, (bool, int)):
        return (ctypes.c_int32 * n)(*([int(bool(flags))] * n))
    if len(flags) != n:
        raise DPError(f"one {what} flag per layer")
    return (ctypes.c_int32 * n)(*[int(bool(f)) for f in flags])


def dp_clipped_grad_sum_noised_store(layers: Sequence, outs: Sequence[torch.Tensor], c,
                                     tensor_ids: Sequence[int], sigma: float, C: float,
                                     B_norm: int, seed: int, step: int, store: torch.Tensor,
                                     accumulate=None, transpose_out=False,
                                     stream=None) -> None:
    """The noised clipped sums from the tiles dp_ghost_norm_linear_store kept
    for the same layers. ``accumulate`` and ``transpose_out`` are a bool or
    one bool per layer."""
    descs = [_layer(l[0], l[1]) for l in layers]
    arr = (dp_linear_t * len(descs))(*descs)
    optrs = (ctypes.c_void_p * len(outs))(*[o.data_ptr() for o in outs])
    tids, acc = _noise_arrays(len(descs), tensor_ids, accumulate)
    tr = _flags(len(descs), transpose_out, "transpose")
    A0 = layers[0][0]
    _check(lib().dp_clipped_grad_sum_noised_store(arr, optrs, tids, acc, tr, len(descs),
                                                  c.data_ptr(), A0.shape[0], A0.shape[1],
                                                  _dtype(A0), float(sigma), float(C),
                                                  int(B_norm), int(seed), int(step),
                                                  store.data_ptr(),
                                                  store.numel() * store.element_size(),
                                                  _stream(stream)),
           "dp_clipped_grad_sum_noised_store")


class LinearGroup:
    """Descriptors of many linear layers of one batch, prepared once.

    Holds the ctypes descriptor array, the output-pointer array and the norm
    workspace so that repeated steps only pass pointers. ``layers`` is a
    sequence of (A, G) or (A, G, algo) with a common B, T and dtype.
    ``bias_grads`` (one fp32 [B, d_out] tensor or None per layer) makes
    ghost_norm also write the layers' per-example bias gradients and count
    their norms (dp_ghost_norm_linear_bias_grouped).
    """

    def __init__(self, layers: Sequence, outs: Optional[Sequence[torch.Tensor]] = None,
                 bias_grads: Optional[Sequence[Optional[torch.Tensor]]] = None):
        L = lib()
        self._tensors = [t for l in layers for t in l[:2]]
        self.n = len(layers)
        self.descs = (dp_linear_t * self.n)(*[_layer(*l) for l in layers])
        A0 = layers[0][0]
        self.B, self.T, self.dt = A0.shape[0], A0.shape[1], _dtype(A0)
        for l in layers:
            if tuple(l[0].shape[:2]) != (self.B, self.T) or _dtype(l[0]) != self.dt:
                raise DPError("all layers of a group share B, T and dtype")
        self._bias = None
        if bias_grads is not None:
            if len(bias_grads) != self.n:
                raise DPError("one bias gradient (or None) per layer")
            for l, g in zip(layers, bias_grads):
                if g is not None and (g.dtype != torch.float32 or not g.is_contiguous()
                                      or tuple(g.shape) != (self.B, l[1].shape[2])):
                    raise DPError("bias gradients must be contiguous fp32 [B, d_out]")
            self._bias_t = list(bias_grads)
            self._bias = (ctypes.c_void_p * self.n)(*[None if g is None else g.data_ptr()
                                                      for g in bias_grads])
        nbytes = L.dp_ghost_norm_linear_bias_workspace(self.descs, self._bias, self.n, self.B,
                                                       self.T, self.dt)
        self.ws = _ws(nbytes, A0.device)
        self._sum_bytes = {}
        self.outs = None
        if outs is not None:
            self.set_outputs(outs)

    def set_outputs(self, outs: Sequence[torch.Tensor]) -> None:
        if len(outs) != self.n:
            raise DPError("one output per layer")
        self._outs = list(outs)
        self.outs = (ctypes.c_void_p * self.n)(*[o.data_ptr() for o in outs])

    def ghost_norm(self, norm2: torch.Tensor, accumulate: bool = False, stream=None):
        _check(lib().dp_ghost_norm_linear_bias_grouped(self.descs, self._bias, self.n, self.B,
                                                       self.T, self.dt, norm2.data_ptr(),
                                                       int(accumulate), self.ws.data_ptr(),
                                                       self.ws.numel(), _stream(stream)),
               "dp_ghost_norm_linear_bias_grouped")
        return norm2

    def clipped_sum(self, c: torch.Tensor, transpose_out: bool = False,
                    accumulate: bool = False, stream=None) -> None:
        if self.outs is None:
            raise DPError("set_outputs() first")
        ws = self._sum_ws(transpose_out, stream)
        _check(lib().dp_clipped_grad_sum_grouped_ws(self.descs, self.outs, self.n, c.data_ptr(),
                                                    self.B, self.T, self.dt, int(transpose_out),
                                                    int(accumulate),
                                                    None if ws is None else ws.data_ptr(),
                                                    0 if ws is None else ws.numel(),
                                                    _stream(stream)),
               "dp_clipped_grad_sum_grouped_ws")

    def _sum_ws(self, transpose_out: bool, stream):
        """The split tail's workspace: every call's own, as calls on other streams
        and replays of a captured one may overlap. Its size is kept per layout."""
        key = bool(transpose_out)
        if key not in self._sum_bytes:
            self._sum_bytes[key] = _split_bytes(self.descs, self.n, self.B, self.T, self.dt, key)
        self._split_ws = None
        nbytes = self._sum_bytes[key]
        ws = _ws(nbytes, self.ws.device, stream) if nbytes else None
        self._split_ws = ws
        return ws

    def clipped_sum_noised(self, c: torch.Tensor, tensor_ids: Sequence[int], sigma: float,
                           C: float, B_norm: int, seed: int, step: int, accumulate=None,
                           transpose_out: bool = False, stream=None) -> None:
        """clipped_sum with the Gaussian mechanism fused (see
        dp_clipped_grad_sum_noised_grouped)."""
        if self.outs is None:
            raise DPError("set_outputs() first")
        key = (tuple(int(t) for t in tensor_ids),
               accumulate if isinstance(accumulate, (bool, int, type(None)))
               else tuple(bool(a) for a in accumulate))
        if getattr(self, "_noise_key", None) != key:
            self._noise_key = key
            self._noise_arr = _noise_arrays(self.n, tensor_ids, accumulate)
        tids, acc = self._noise_arr
        L = lib()
        ws = self._sum_ws(transpose_out, stream)
        _check(L.dp_clipped_grad_sum_noised_grouped_ws(self.descs, self.outs, tids, acc, self.n,
                                                       c.data_ptr(), self.B, self.T, self.dt,
                                                       int(transpose_out), float(sigma), float(C),
                                                       int(B_norm), int(seed), int(step),
                                                       None if ws is None else ws.data_ptr(),
                                                       0 if ws is None else ws.numel(),
                                                       _stream(stream)),
               "dp_clipped_grad_sum_noised_grouped_ws")

    def store_bytes(self) -> int:
        """Bytes of the per-example gradient store for this group (0: the
        store form does not apply; see dp_grad_store_bytes)."""
        return lib().dp_grad_store_bytes(self.descs, self.n, self.B, self.T, self.dt)

    def ghost_norm_store(self, norm2: torch.Tensor, store: torch.Tensor,
                         accumulate: bool = False, stream=None) -> torch.Tensor:
        """Direct norms of every layer, the examples' gradient tiles into store."""
        _check(lib().dp_ghost_norm_linear_store(self.descs, self.n, self.B, self.T, self.dt,
                                                norm2.data_ptr(), int(accumulate),
                                                store.data_ptr(),
                                                store.numel() * store.element_size(),
                                                _stream(stream)),
               "dp_ghost_norm_linear_store")
        return norm2

    def clipped_sum_noised_store(self, c: torch.Tensor, store: torch.Tensor,
                                 tensor_ids: Sequence[int], sigma: float, C: float, B_norm: int,
                                 seed: int, step: int, accumulate=None, transpose_out=False,
                                 stream=None) -> None:
        """clipped_sum_noised from the tiles ghost_norm_store kept;
        ``transpose_out`` is a bool or one bool per layer."""
        if self.outs is None:
            raise DPError("set_outputs() first")
        key = (tuple(int(t) for t in tensor_ids),
               accumulate if isinstance(accumulate, (bool, int, type(None)))
               else tuple(bool(a) for a in accumulate),
               transpose_out if isinstance(transpose_out, (bool, int))
               else tuple(bool(t) for t in transpose_out))
        if getattr(self, "_store_key", None) != key:
            self._store_key = key
            self._store_arr = (*_noise_arrays(self.n, tensor_ids, accumulate),
                               _flags(self.n, transpose_out, "transpose"))
        tids, acc, tr = self._store_arr
        _check(lib().dp_clipped_grad_sum_noised_store(self.descs, self.outs, tids, acc, tr,
                                                      self.n, c.data_ptr(), self.B, self.T,
                                                      self.dt, float(sigma), float(C),
                                                      int(B_norm), int(seed), int(step),
                                                      store.data_ptr(),
                                                      store.numel() * store.element_size(),
                                                      _stream(stream)),
               "dp_clipped_grad_sum_noised_store")
