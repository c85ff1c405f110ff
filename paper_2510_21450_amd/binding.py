"""Python binding: one function per entry point of include/pararnn.h, same names without the prefix.
Argument marshalling only: by the native module _host (csrc/host_binding.cpp) for the calls of a model's
inner loop, by ctypes for the rest."""
from __future__ import annotations

import ctypes
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_PKG, "libpararnn.so")

CELLS = {"gru_diag": 0, "lstm_diag": 1, "tanh_dense": 2, "linear_diag": 3, "paralstm_diag": 4}
DTYPES = {torch.float32: 0, torch.bfloat16: 1}
STATUS = {0: "OK", 1: "NOT_CONVERGED", 2: "INVALID_ARG", 3: "WORKSPACE_TOO_SMALL", 4: "HIP_ERROR",
          5: "NONFINITE", 6: "UNSUPPORTED", 7: "INTERNAL"}

if not os.path.exists(_LIB_PATH):
    raise ImportError(f"{_LIB_PATH} is missing: build it with `python -m paper_2510_21450_amd.build` "
                      "(there is no CPU fallback)")

_lib = ctypes.CDLL(_LIB_PATH)
try:
    from . import _host
except ImportError as e:
    raise ImportError(f"the native binding module beside {_LIB_PATH} is missing or unusable ({e}): build it with "
                      "`python -m paper_2510_21450_amd.build`") from e
for _name in ("pararnn_input_projection", "pararnn_residual_norm", "pararnn_set_dense_jacobian", "pararnn_device_info", "pararnn_set_dense_products", "pararnn_solve_plan", "pararnn_affine_scan_workspace_bytes"):
    if not hasattr(_lib, _name):
        raise ImportError(f"{_LIB_PATH} is older than this binding ({_name} is missing): rebuild it with "
                          "`python -m paper_2510_21450_amd.build`")
_vp, _i, _f, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
_lib.pararnn_status_string.restype = ctypes.c_char_p
_lib.pararnn_status_string.argtypes = [_i]
_lib.pararnn_version.restype = _i
_lib.pararnn_device_info.restype = _i
_lib.pararnn_device_info.argtypes = [ctypes.POINTER(ctypes.c_int), _i]
_lib.pararnn_set_tile.argtypes = [_i] * 4
_lib.pararnn_set_tile.restype = _i
_lib.pararnn_cell_gates.argtypes = [_i]
_lib.pararnn_cell_state.argtypes = [_i]
_lib.pararnn_workspace_bytes.restype = _sz
_lib.pararnn_workspace_bytes.argtypes = [_i] * 6
_lib.pararnn_workspace_bytes_fused.restype = _sz
_lib.pararnn_workspace_bytes_fused.argtypes = [_i] * 6
_lib.pararnn_set_fused.argtypes = [_i]
_lib.pararnn_set_fused_tail.argtypes = [_i]
_lib.pararnn_set_workspace_reuse.argtypes = [_i]
_lib.pararnn_set_staging.argtypes = [_i]
_lib.pararnn_set_streaming.argtypes = [_i]
_lib.pararnn_set_dense_products.argtypes = [_i]
_lib.pararnn_set_fused_head.argtypes = [_i]
_lib.pararnn_solve_plan.restype = _i
_lib.pararnn_solve_plan.argtypes = [ctypes.c_float, _i, ctypes.POINTER(ctypes.c_int), _i]
class _SolveOptions(ctypes.Structure):
    _fields_ = [("first_block", ctypes.c_int), ("fused", ctypes.c_int)]


_lib.pararnn_forward_ex.restype = _i
_lib.pararnn_forward_ex.argtypes = [_i, _i, _vp, _vp, _vp, _i, _i, _i, _f, _i, _vp, _vp, _vp, _vp, _sz, _vp,
                                    ctypes.POINTER(_SolveOptions)]
_lib.pararnn_workspace_bytes_ex.restype = _sz
_lib.pararnn_workspace_bytes_ex.argtypes = [_i, _i, _i, _i, _i, ctypes.POINTER(_SolveOptions)]
_lib.pararnn_solve_plan_ex.restype = _i
_lib.pararnn_solve_plan_ex.argtypes = [ctypes.c_float, _i, ctypes.POINTER(_SolveOptions), ctypes.POINTER(ctypes.c_int), _i]
_lib.pararnn_forward_noalloc.restype = _i
_lib.pararnn_forward_noalloc.argtypes = [_i, _i, _vp, _vp, _vp, _i, _i, _i, _f, _i, _vp, _vp, _vp, _vp]
_lib.pararnn_dense_chunk_products.restype = _i
_lib.pararnn_dense_chunk_products.argtypes = [_vp, _vp, _i, _i, _i, _vp, _vp, _sz, _vp]
_lib.pararnn_affine_scan.restype = _i
_lib.pararnn_affine_scan_workspace_bytes.restype = _sz
_lib.pararnn_affine_scan_workspace_bytes.argtypes = [_i] * 5
_lib.pararnn_affine_scan.argtypes = [_i, _i, _vp, _vp, _i, _i, _i, _vp, _vp, _sz, _vp]


_RES_ARGS = [_i, _vp, _vp, _vp, _vp, _i, _i, _i, _vp, _vp]
_lib.pararnn_residual_norm.restype = _i
_lib.pararnn_residual_norm.argtypes = [_i] + _RES_ARGS


class _BuiltinCell:
    """Entry points of one built-in cell: the pararnn_* functions with the cell number bound."""

    def __init__(self, name):
        self.name = name
        c = CELLS[name]
        self.G, self.S = _lib.pararnn_cell_gates(c), _lib.pararnn_cell_state(c)
        self.what = "pararnn"
        self.ws = lambda *a: _lib.pararnn_workspace_bytes(c, *a)
        self.ws_fused = lambda *a: _lib.pararnn_workspace_bytes_fused(c, *a)
        self.host = _host.builtin_cell(c, self.what)
        self.res = lambda *a: _lib.pararnn_residual_norm(c, *a)


class UserCell:
    """A cell from a library built with PARARNN_DEFINE_CELL(Cell, name) (include/pararnn_cell.h):
    pass the object wherever the functions of this module take a cell name."""

    def __init__(self, lib_path: str, name: str):
        if not os.path.exists(lib_path):
            raise ImportError(f"{lib_path} is missing: build it with `python -m paper_2510_21450_amd.build --cell ...`")
        self.name, self.what = name, name
        self._lib = lib = ctypes.CDLL(lib_path)
        f = lambda s: getattr(lib, f"{name}_{s}")
        self.G, self.S, self.param_rows = f("gates")(), f("state")(), f("param_rows")()
        self.ws, self.ws_fused = f("workspace_bytes"), f("workspace_bytes_fused")
        self.ws.restype = self.ws_fused.restype = _sz
        self.ws.argtypes = self.ws_fused.argtypes = [_i] * 5
        address = lambda s: ctypes.cast(f(s), _vp).value
        parts = address("workspace_parts") if hasattr(lib, f"{name}_workspace_parts") else 0
        self.host = _host.library_cell(name, self.G, self.S, address("workspace_bytes"), address("workspace_bytes_fused"),
                                       address("forward"), address("backward"), parts)
        self.res = f("residual_norm")
        self.res.restype, self.res.argtypes = _i, _RES_ARGS


_builtin = {}


def _api(cell):
    if isinstance(cell, UserCell):
        return cell
    if cell not in _builtin:
        _builtin[cell] = _BuiltinCell(cell)
    return _builtin[cell]


def example_cell(name: str) -> UserCell:
    """One of the example cells shipped under user_cells/ ("gru_softsign", "gru_sigmoid_identity_tanh",
    "gru_sigmoid_softsign_identity", "gru_sigmoid_tanh_softsign", "rot_tanh", "tri_tanh", "quad_tanh")."""
    return UserCell(os.path.join(_PKG, f"libpararnn_{name}.so"), name)


def set_tile(vec: int = 0, ll: int = 0, c: int = 0, w: int = 0) -> None:
    """pararnn_set_tile: force a compiled tile shape (vec = 0: automatic)."""
    _raise(_lib.pararnn_set_tile(vec, ll, c, w), "pararnn_set_tile")


def set_dense_products(mode: int = 0) -> None:
    """pararnn_set_dense_products: 0 fp32 Jacobian products (default), 1 three bf16 terms, 2 one bf16 term."""
    _raise(_lib.pararnn_set_dense_products(int(mode)), "pararnn_set_dense_products")


def device_info() -> dict:
    """pararnn_device_info as a dict (None where the runtime gives no answer)."""
    buf = (ctypes.c_int * 8)()
    n = _lib.pararnn_device_info(buf, 8)
    if n < 6:
        raise RuntimeError("pararnn_device_info failed")
    keys = ("compute_units", "clock_khz", "memory_clock_khz", "memory_bus_bits", "l2_bytes", "lds_bytes_per_workgroup")
    return {k: (int(buf[i]) if buf[i] >= 0 else None) for i, k in enumerate(keys)}


def set_dense_jacobian(mode: int = 0) -> None:
    """pararnn_set_dense_jacobian: 0 the full Jacobian (Newton, default), 1 its diagonal (quasi-Newton)."""
    _raise(_lib.pararnn_set_dense_jacobian(int(mode)), "pararnn_set_dense_jacobian")


def set_dense_tail(mode: int = 1) -> None:
    """pararnn_set_dense_tail: 1 launches per phase for six iterations, then one persistent launch (default);
    0 launches per phase throughout; 2 the persistent launch from the start."""
    _raise(_lib.pararnn_set_dense_tail(int(mode)), "pararnn_set_dense_tail")


def set_dense_substitution(enable: bool = True) -> None:
    """pararnn_set_dense_substitution: solve linear systems by forward substitution where it is faster (default), or
    always by the chunked scan."""
    _raise(_lib.pararnn_set_dense_substitution(int(enable)), "pararnn_set_dense_substitution")


def dense_chunk() -> int:
    return _lib.pararnn_dense_chunk()


def dense_chunk_products(W, d, out=None, stream=None):
    """pararnn_dense_chunk_products.  W [H][H], d [B][L][H] -> A [B][n_c][H][H]
    (chunks 1 .. n_c-2 written, the rest zero)."""
    B, L, H = d.shape
    _check(W, "W", torch.float32, (H, H))
    _check(d, "d", torch.float32)
    n_c = (L + dense_chunk() - 1) // dense_chunk()
    A = torch.zeros((B, n_c, H, H), dtype=torch.float32, device=d.device) if out is None else out
    ws = torch.empty(256, dtype=torch.uint8, device=d.device)
    code = _lib.pararnn_dense_chunk_products(_ptr(W), _ptr(d), B, L, H, _ptr(A), _ptr(ws), ws.numel(), _stream(stream))
    _raise(code, "pararnn_dense_chunk_products")
    return A


def lib_path() -> str:
    return _LIB_PATH


def version() -> int:
    return _lib.pararnn_version()


def status_string(code: int) -> str:
    return _lib.pararnn_status_string(code).decode()


def cell_dims(cell):
    """(gates G, state values S) of a cell (a built-in cell's name or a UserCell)."""
    a = _api(cell)
    return a.G, a.S


def workspace_bytes(cell, dtype, B: int, L: int, H: int, backward: bool = False) -> int:
    return _api(cell).ws(DTYPES[dtype], B, L, H, int(backward))


def workspace_bytes_fused(cell, dtype, B: int, L: int, H: int, n_iters: int) -> int:
    return _api(cell).ws_fused(DTYPES[dtype], B, L, H, n_iters)


def set_spin_limit(polls: int = 0) -> None:
    """pararnn_set_spin_limit: polls of a predecessor's carry record before a tile gives up (0 = default)."""
    _lib.pararnn_set_spin_limit.argtypes = [ctypes.c_uint]
    _raise(_lib.pararnn_set_spin_limit(int(polls)), "pararnn_set_spin_limit")


def set_fused(enable: bool = True) -> None:
    """pararnn_set_fused: allow (default) or forbid the fused multi-iteration launches."""
    _raise(_lib.pararnn_set_fused(int(enable)), "pararnn_set_fused")


def set_staging(enable: bool = True) -> None:
    """pararnn_set_staging: allow (default) or forbid the kernel variants that stage their inputs through LDS."""
    _raise(_lib.pararnn_set_staging(int(enable)), "pararnn_set_staging")


def solve_plan(tol: float, max_iter: int):
    """pararnn_solve_plan: Newton iterations per launch of a solve with the current settings."""
    buf = (ctypes.c_int * max(1, max_iter))()
    n = _lib.pararnn_solve_plan(float(tol), int(max_iter), buf, max(1, max_iter))
    if n < 0:
        raise ValueError("pararnn_solve_plan: invalid arguments")
    return [buf[i] for i in range(n)]


def solve_without_blocks(cell, dtype, B: int, L: int, H: int, tol: float, max_iter: int) -> bool:
    """pararnn_solve_without_blocks (built-in cells): whether `forward` solves this problem in one launch without the blocks
    of `solve_plan`, one workgroup per group of channels."""
    r = _lib.pararnn_solve_without_blocks(CELLS[cell], DTYPES[dtype], B, L, H, ctypes.c_float(tol), int(max_iter))
    if r < 0:
        raise ValueError("pararnn_solve_without_blocks: invalid arguments")
    return bool(r)


def solve_walked(cell, dtype, B: int, L: int, H: int, tol: float, max_iter: int) -> bool:
    """pararnn_solve_walked (built-in cells): whether `forward` solves this problem in one launch without the blocks of
    `solve_plan`, every wave walking the sequences of a group of channels."""
    r = _lib.pararnn_solve_walked(CELLS[cell], DTYPES[dtype], B, L, H, ctypes.c_float(tol), int(max_iter))
    if r < 0:
        raise ValueError("pararnn_solve_walked: invalid arguments")
    return bool(r)


def set_streaming(mode: int = 0) -> None:
    """pararnn_set_streaming: streamed tile accesses of the memory-bound kernels chosen by size (0, default),
    never (1) or always (2)."""
    _raise(_lib.pararnn_set_streaming(int(mode)), "pararnn_set_streaming")


def set_workspace_reuse(enable: bool = False) -> None:
    """pararnn_set_workspace_reuse: the caller's promise that nothing else writes to a workspace between the
    library's calls on it; the carry records are then not cleared again for a call of the same layout."""
    _raise(_lib.pararnn_set_workspace_reuse(int(enable)), "pararnn_set_workspace_reuse")


def release_workspaces() -> int:
    """Give what `forward`, `backward` and the autograd functions keep of their workspaces between calls (at most 16 and a
    thirty-second of the memory per device) back to torch's allocator; returns their bytes.  The allocator gets them back by
    itself before it takes more memory from the device."""
    return _host.release_workspaces()


def set_fused_tail(enable: bool = True) -> None:
    """pararnn_set_fused_tail: the blocks after a solve's first launch share one persistent launch (default)
    or are launches of their own."""
    _raise(_lib.pararnn_set_fused_tail(int(enable)), "pararnn_set_fused_tail")


def set_fused_head(n_iters: int = 5) -> None:
    """pararnn_set_fused_head: iterations a solve to a tolerance runs in its first launch (0 = none)."""
    _raise(_lib.pararnn_set_fused_head(int(n_iters)), "pararnn_set_fused_head")


def _ptr(t):
    return None if t is None else t.data_ptr()


def _check(t, name, dtype, shape=None):
    if not t.is_cuda:
        raise ValueError(f"{name} must be a CUDA tensor")
    if t.dtype != dtype:
        raise ValueError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} must have shape {tuple(shape)}, got {tuple(t.shape)}")


def _stream(stream):
    s = torch.cuda.current_stream() if stream is None else stream
    return s.cuda_stream


def _raw_stream(stream):
    """The stream's handle for the native module, which takes the current stream for None itself."""
    return None if stream is None else stream.cuda_stream


def _workspace(nbytes, device, workspace):
    if workspace is None:
        workspace = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=device)
    return workspace


def _raise(code, what):
    if code != 0:
        raise RuntimeError(f"{what} failed: {status_string(code)} ({code})")


def forward(cell, params, u, h0=None, tol: float = 1e-6, max_iter: int = 64, trace: bool = False,
            workspace=None, stream=None, out=None):
    """pararnn_forward (or <name>_forward of a UserCell).  u [B][L][G][H] (fp32 or bf16), params fp32.
    Returns (h, iters, delta_trace): iters is a DEVICE int32[2] tensor
    {iterations, status} (no synchronisation happens here), delta_trace a
    device float[max_iter] tensor or None."""
    return _host.forward(_api(cell).host, params, u, h0, tol, max_iter, trace, workspace, _raw_stream(stream), out)


def forward_ex(cell, params, u, h0=None, tol: float = 1e-6, max_iter: int = 64, first_block: int = -1, fused: int = -1,
               trace: bool = False, workspace=None, stream=None, out=None):
    """pararnn_forward_ex (built-in cells): `forward` with the size of the first fused block and the
    fused switch as arguments of the call (-1 = the library's setting).  Same return values."""
    G, S = cell_dims(cell)
    B, L, Gu, H = u.shape
    dt = u.dtype
    _check(u, "u", dt, (B, L, G, H))
    _check(params, "params", torch.float32)
    if h0 is not None:
        _check(h0, "h0", dt, (B, S, H))
    h = torch.empty((B, L, S, H), dtype=dt, device=u.device) if out is None else out
    _check(h, "h", dt, (B, L, S, H))
    iters = torch.empty(2, dtype=torch.int32, device=u.device)
    tr = torch.zeros(max(max_iter, 1), dtype=torch.float32, device=u.device) if trace else None
    opt = _SolveOptions(int(first_block), int(fused))
    need = max(_lib.pararnn_workspace_bytes_ex(CELLS[cell], DTYPES[dt], B, L, H, ctypes.byref(opt)),
               workspace_bytes_fused(cell, dt, B, L, H, max_iter) if tol < 0 else 0)
    ws = _workspace(need, u.device, workspace)
    code = _lib.pararnn_forward_ex(CELLS[cell], DTYPES[dt], _ptr(params), _ptr(u), _ptr(h0), B, L, H, tol, max_iter,
                                   _ptr(h), _ptr(iters), _ptr(tr), _ptr(ws), ws.numel(), _stream(stream),
                                   ctypes.byref(opt))
    _raise(code, "pararnn_forward_ex")
    return h, iters, tr


def solve_plan_ex(tol: float, max_iter: int, first_block: int = -1, fused: int = -1):
    """pararnn_solve_plan_ex: Newton iterations per launch of a solve with the given options."""
    buf = (ctypes.c_int * max(1, max_iter))()
    opt = _SolveOptions(int(first_block), int(fused))
    n = _lib.pararnn_solve_plan_ex(float(tol), int(max_iter), ctypes.byref(opt), buf, max(1, max_iter))
    if n < 0:
        raise ValueError("pararnn_solve_plan_ex: invalid arguments")
    return [buf[i] for i in range(n)]


def forward_noalloc(cell, params, u, h0, tol, max_iter, out, iters, delta_trace=None, stream=None):
    """pararnn_forward_noalloc (built-in cells): the solve of `forward` on the library's static
    scratch array.  Nothing is allocated here either: `out` [B][L][S][H], `iters` (device int32[2])
    and, if wanted, `delta_trace` (device float[max_iter]) are the caller's.  Returns the C status
    code (0 = enqueued); a problem too large for the array gives WORKSPACE_TOO_SMALL (3)."""
    G, S = cell_dims(cell)
    B, L, Gu, H = u.shape
    dt = u.dtype
    _check(u, "u", dt, (B, L, G, H))
    _check(params, "params", torch.float32)
    if h0 is not None:
        _check(h0, "h0", dt, (B, S, H))
    _check(out, "h", dt, (B, L, S, H))
    _check(iters, "iters", torch.int32, (2,))
    if delta_trace is not None:
        _check(delta_trace, "delta_trace", torch.float32, (max(max_iter, 1),))
    return _lib.pararnn_forward_noalloc(CELLS[cell], DTYPES[dt], _ptr(params), _ptr(u), _ptr(h0), B, L, H, tol,
                                        max_iter, _ptr(out), _ptr(iters), _ptr(delta_trace), _stream(stream))


def backward(cell, params, u, h0, h, dL_dh, want_dh0: bool = True, workspace=None, stream=None, out=None):
    """pararnn_backward.  Returns (dL_du, dL_dparams, dL_dh0 or None); `out`
    may hold a preallocated (dL_du, dL_dparams, dL_dh0) triple."""
    return _host.backward(_api(cell).host, params, u, h0, h, dL_dh, want_dh0, workspace, _raw_stream(stream),
                          *(out if out is not None else (None, None, None)))


def residual_norm(cell, params, u, h0, h, stream=None, out=None):
    """pararnn_residual_norm: max |h_l - f(h_{l-1}, u_l)| of the given states, as a device float[1]."""
    G, S = cell_dims(cell)
    B, L, Gu, H = u.shape
    dt = u.dtype
    _check(u, "u", dt, (B, L, G, H))
    _check(params, "params", torch.float32)
    _check(h, "h", dt, (B, L, S, H))
    if h0 is not None:
        _check(h0, "h0", dt, (B, S, H))
    if out is None:
        out = torch.empty(1, dtype=torch.float32, device=u.device)
    _check(out, "out", torch.float32, (1,))
    api = _api(cell)
    code = api.res(DTYPES[dt], _ptr(params), _ptr(u), _ptr(h0), _ptr(h), B, L, H, _ptr(out), _stream(stream))
    _raise(code, f"{api.what}_residual_norm")
    return out


_lib.pararnn_input_projection_workspace_bytes.restype = _sz
_lib.pararnn_input_projection_workspace_bytes.argtypes = [_i] * 7


def input_projection_workspace_bytes(dtype, B: int, L: int, H: int, G: int, n_heads: int = 1, backward: bool = False) -> int:
    return _lib.pararnn_input_projection_workspace_bytes(DTYPES[dtype], B, L, H, G, n_heads, int(backward))


def input_projection(x, Wx, bias=None, n_heads: int = 1, workspace=None, stream=None, out=None):
    """pararnn_input_projection.  x [B][L][H], Wx fp32 [G][H][H / n_heads], bias fp32 [G][H] or None
    -> u [B][L][G][H] of x's dtype."""
    return _host.input_projection(x, Wx, bias, n_heads, workspace, _raw_stream(stream), out)


def input_projection_backward(x, Wx, du, n_heads: int = 1, want_dx: bool = True, want_dw: bool = True,
                              want_dbias: bool = True, workspace=None, stream=None):
    """pararnn_input_projection_backward.  Returns (dx, dWx, dbias); entries not wanted are None."""
    return _host.input_projection_backward(x, Wx, du, n_heads, want_dx, want_dw, want_dbias, workspace, _raw_stream(stream))


def affine_scan(J, r, reverse: bool = False, workspace=None, stream=None):
    """pararnn_affine_scan.  J [B][L][H] (diagonal) or [B][L][S][S][H] (blocks,
    S = 2, 3, 4); r [B][L][S][H] or [B][L][H].  Returns delta with r's shape."""
    B, L = r.shape[0], r.shape[1]
    H = r.shape[-1]
    if J.dim() == 3:
        kind = 0
        _check(J, "J", torch.float32, (B, L, H))
    else:
        S = J.shape[2]
        if J.dim() != 5 or S not in (2, 3, 4):
            raise ValueError("J must be [B][L][H] or [B][L][S][S][H] with S in 2..4")
        kind = S - 1
        _check(J, "J", torch.float32, (B, L, S, S, H))
    _check(r, "r", torch.float32)
    delta = torch.empty_like(r)
    ws = _workspace(_lib.pararnn_affine_scan_workspace_bytes(kind, int(reverse), B, L, H), r.device, workspace)
    code = _lib.pararnn_affine_scan(kind, int(reverse), _ptr(J), _ptr(r), B, L, H, _ptr(delta), _ptr(ws),
                                    ws.numel(), _stream(stream))
    _raise(code, "pararnn_affine_scan")
    return delta
