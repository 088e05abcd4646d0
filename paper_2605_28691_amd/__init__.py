"""MI355X-native Skiparse-2D attention: thin Python binding over the C ABI in ``include/skiparse.h``.

Argument marshalling only.  Tensors are ``torch`` CUDA(HIP) tensors used purely as device memory; every step of
the path runs in the library's own kernels on the current torch stream.  There is no CPU fallback: without the
built library, or on a bad argument, a call raises.
"""
from __future__ import annotations

import ctypes
import functools
import importlib
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libskiparse.so")

TOKEN, GROUP = 0, 1
BF16, FP32, FP8_E4M3 = 0, 1, 2
FUSED = 1
PAD = 2
PATTERNS = {"token": TOKEN, "group": GROUP}
OUT_LAYOUTS = {"same": 0, "other": 1, "original": 2}
_DTYPES = {torch.bfloat16: BF16, torch.float32: FP32, torch.uint8: FP8_E4M3, torch.float8_e4m3fn: FP8_E4M3}

_lib = None


class SkiparseError(RuntimeError):
    def __init__(self, code: int, what: str):
        msg = lib().skiparse_strerror(code).decode()
        extra = f" [hipError {lib().skiparse_last_hip_error()}]" if code == -5 else ""
        super().__init__(f"{what}: {msg} (code {code}){extra}")
        self.code = code


def lib() -> ctypes.CDLL:
    """Loads libskiparse.so (built by ``paper_2605_28691_amd.build.build()``); raises if it is missing."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise RuntimeError(
                f"{_LIB_PATH} is missing: build it first (python -m paper_2605_28691_amd.build); there is no fallback path"
            )
        L = ctypes.CDLL(_LIB_PATH)
        i, vp, f, u, sz = ctypes.c_int, ctypes.c_void_p, ctypes.c_float, ctypes.c_uint, ctypes.c_size_t
        L.skiparse_permute.restype = i
        L.skiparse_permute.argtypes = [vp, vp] + [i] * 9 + [vp]
        L.skiparse_unpermute.restype = i
        L.skiparse_unpermute.argtypes = [vp, vp] + [i] * 9 + [vp]
        L.skiparse_switch_pattern.restype = i
        L.skiparse_switch_pattern.argtypes = [vp, vp] + [i] * 9 + [vp]
        L.skiparse_ssp_pack.restype = i
        L.skiparse_ssp_pack.argtypes = [vp, vp] + [i] * 9 + [vp]
        L.skiparse_ssp_unpack.restype = i
        L.skiparse_ssp_unpack.argtypes = [vp, vp] + [i] * 9 + [vp]
        L.dense_attn_fwd.restype = i
        L.dense_attn_fwd.argtypes = [vp] * 4 + [i] * 6 + [f, i, vp]
        L.skiparse_attn_fwd.restype = i
        L.skiparse_attn_fwd.argtypes = [vp] * 4 + [i] * 8 + [f, i, u, vp, sz, vp]
        L.skiparse_attn_fwd_sparse.restype = i
        L.skiparse_attn_fwd_sparse.argtypes = [vp] * 4 + [i] * 9 + [f, i, vp]
        L.skiparse_lse_bytes.restype = sz
        L.skiparse_lse_bytes.argtypes = [i] * 8 + [u]
        L.skiparse_attn_fwd_lse.restype = i
        L.skiparse_attn_fwd_lse.argtypes = [vp] * 5 + [i] * 8 + [f, i, u, vp]
        L.skiparse_bwd_workspace_bytes.restype = sz
        L.skiparse_bwd_workspace_bytes.argtypes = [i] * 8 + [u]
        L.skiparse_bwd_walk_workspace_bytes.restype = sz
        L.skiparse_bwd_walk_workspace_bytes.argtypes = [i] * 8 + [u]
        L.skiparse_attn_bwd.restype = i
        L.skiparse_attn_bwd.argtypes = [vp] * 9 + [i] * 8 + [f, i, u, vp, sz, vp]
        L.skiparse_attn_bwd_static.restype = i
        L.skiparse_attn_bwd_static.argtypes = [vp] * 9 + [i] * 8 + [f, i, u, vp]
        L.skiparse_static_scratch_bytes.restype = sz
        L.skiparse_static_scratch_bytes.argtypes = []
        L.skiparse_workspace_bytes.restype = sz
        L.skiparse_workspace_bytes.argtypes = [i] * 8 + [u]
        L.skiparse_quantize_fp8_ex.restype = i
        L.skiparse_quantize_fp8_ex.argtypes = [vp, vp, vp] + [i] * 8 + [u, vp]
        L.skiparse_attn_fwd_fp8_ex.restype = i
        L.skiparse_attn_fwd_fp8_ex.argtypes = [vp] * 7 + [i] * 8 + [f, u, vp]
        L.skiparse_quantize_fp8.restype = i
        L.skiparse_quantize_fp8.argtypes = [vp, vp, vp] + [i] * 8 + [vp]
        L.skiparse_attn_fwd_fp8.restype = i
        L.skiparse_attn_fwd_fp8.argtypes = [vp] * 7 + [i] * 8 + [f, vp]
        L.skiparse_strerror.restype = ctypes.c_char_p
        L.skiparse_strerror.argtypes = [i]
        L.skiparse_last_hip_error.restype = i
        L.skiparse_last_hip_error.argtypes = []
        _bind(L)
        _lib = L
    return _lib


# A small call is bound by what it costs to issue it, so no Stream object is made for it.  torch hands out the bare handle under private names
# only; where a release has no such names the Stream object serves.
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_get_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream() -> int:
    """Handle of torch's current stream on the current device."""
    if _raw_stream is None or _get_device is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_get_device())


def _forked() -> None:
    """The bare handle is given out without a look at where: in a forked child torch's public call decides, which refuses the GPU to the
    child of a process that has used it."""
    global _raw_stream
    _raw_stream = None


os.register_at_fork(after_in_child=_forked)


def _dev(t: torch.Tensor, name: str) -> int:
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError(f"{name} must be a contiguous device tensor")
    return t.data_ptr()


def _check(code: int, what: str) -> None:
    if code != 0:
        raise SkiparseError(code, what)


# Where the tensors of a call stand in the C function's arguments, and what they are called when one is refused.
_QKVO = ((0, "q"), (1, "k"), (2, "v"), (3, "out"))
_TENSORS = {
    "skiparse_permute": ((0, "x"), (1, "out")),
    "skiparse_unpermute": ((0, "y"), (1, "out")),
    "skiparse_switch_pattern": ((0, "y"), (1, "out")),
    "skiparse_ssp_pack": ((0, "x"), (1, "out")),
    "skiparse_ssp_unpack": ((0, "recv"), (1, "out")),
    "dense_attn_fwd": _QKVO,
    "skiparse_attn_fwd": (*_QKVO, (15, "workspace")),
    "skiparse_attn_fwd_sparse": _QKVO,
    "skiparse_attn_fwd_lse": (*_QKVO, (4, "lse")),
    "skiparse_attn_bwd": (*_QKVO, (4, "dout"), (5, "lse"), (6, "dq"), (7, "dk"), (8, "dv"), (20, "workspace")),
    "skiparse_attn_bwd_static": (*_QKVO, (4, "dout"), (5, "lse"), (6, "dq"), (7, "dk"), (8, "dv")),
    "skiparse_quantize_fp8_ex": ((0, "x"), (1, "x8"), (2, "scales")),
    "skiparse_attn_fwd_fp8_ex": ((0, "q8"), (1, "k8"), (2, "v8"), (3, "sq"), (4, "sk"), (5, "sv"), (6, "out")),
}


def _failed(code: int, name: str) -> None:
    _check(code, name.removesuffix("_ex"))


def _general(name: str, *args) -> None:
    """The call by way of ctypes, which takes every integer-like argument and names what it refuses."""
    args = list(args)
    for i, what in _TENSORS[name]:
        if not (args[i] is None and (name, what) == ("skiparse_attn_fwd", "workspace")):  # the fused form needs none
            args[i] = _dev(args[i], what)
    _failed(getattr(lib(), name)(*args), name)


# The entry points themselves: by ctypes until the library is opened, then natively marshalled where there is a module for this Python and
# this torch.  The module is imported then and not with the package, so that a process that builds first gets what it has built.
for _name in _TENSORS:
    globals()["_" + _name] = functools.partial(_general, _name)


def _torch_build() -> str:
    """Which torch this is: the module reads tensors by the layout in the headers that it was built with."""
    return f"{torch.__version__} {torch.version.git_version}"


def _bind(L: ctypes.CDLL) -> None:
    """Looks for the module, and hands it the functions of the library that has been opened."""
    global _marshal
    try:
        native = importlib.import_module(__name__ + "._marshal")
    except ImportError:
        native = None
    if native is not None and getattr(native, "BUILT_FOR", None) != _torch_build():
        native = None
    if native is not None:
        native.set_up(_general, _failed)
        for name in _TENSORS:
            native.bind(name, ctypes.cast(getattr(L, name), ctypes.c_void_p).value)
            globals()["_" + name] = getattr(native, name)
    _marshal = native


def __getattr__(name: str):
    if name == "_marshal":  # the native module, or None: known once the library is open
        lib()
        return globals()[name]
    raise AttributeError(f"module {__name__!r} has no attribute {name!r}")


def _dims(x: torch.Tensor, T: int, H: int, W: int):
    B, N, heads, D = x.shape
    if N != T * H * W:
        raise ValueError("token axis does not match T*H*W")
    return B, heads, D


def skiparse_permute(x: torch.Tensor, T: int, H: int, W: int, s: int, pattern: str, out: torch.Tensor | None = None):
    """[B][N][heads][D] -> [s*s*B][N/s^2][heads][D] (original -> sparse layout), bit-exact row gather."""
    B, heads, D = _dims(x, T, H, W)
    if out is None:
        out = torch.empty((s * s * B, (T * H * W) // (s * s), heads, D), dtype=x.dtype, device=x.device)
    _skiparse_permute(x, out, B, heads, T, H, W, D, s, PATTERNS[pattern], _DTYPES[x.dtype], _stream())
    return out


def skiparse_unpermute(y: torch.Tensor, T: int, H: int, W: int, s: int, pattern: str, out: torch.Tensor | None = None):
    """[s*s*B][N/s^2][heads][D] -> [B][N][heads][D] (sparse -> original layout)."""
    SB, Nsub, heads, D = y.shape
    B = SB // (s * s)
    if SB != B * s * s or Nsub * s * s != T * H * W:
        raise ValueError("sparse-layout shape does not match the grid")
    if out is None:
        out = torch.empty((B, T * H * W, heads, D), dtype=y.dtype, device=y.device)
    _skiparse_unpermute(y, out, B, heads, T, H, W, D, s, PATTERNS[pattern], _DTYPES[y.dtype], _stream())
    return out


def skiparse_switch_pattern(y: torch.Tensor, T: int, H: int, W: int, s: int, from_pattern: str, out: torch.Tensor | None = None):
    """Sparse layout of `from_pattern` -> sparse layout of the other pattern, one row move per token."""
    SB, Nsub, heads, D = y.shape
    B = SB // (s * s)
    if SB != B * s * s or Nsub * s * s != T * H * W:
        raise ValueError("sparse-layout shape does not match the grid")
    if out is None:
        out = torch.empty_like(y)
    _skiparse_switch_pattern(y, out, B, heads, T, H, W, D, s, PATTERNS[from_pattern], _DTYPES[y.dtype], _stream())
    return out


def skiparse_ssp_pack(x: torch.Tensor, T: int, H: int, W: int, s: int, group_size: int, out: torch.Tensor | None = None):
    """One rank's shard [G*b][T*(H/s)*(W/s)][heads][D] (G = s*s/group_size subsequences, batch fastest) -> the all-to-all send buffer
    [group_size][G][G*b][T*(H/s^2)*(W/s^2)][heads][D] of Sparse Sequence Parallelism (chunk r is for rank r)."""
    Bl, n_local, heads, D = x.shape
    G = (s * s) // group_size
    if G < 1 or G * group_size != s * s or Bl % G or n_local * s * s != T * H * W:
        raise ValueError("shard shape does not match the grid and the group")
    if out is None:
        out = torch.empty((group_size, G, Bl, n_local // (s * s), heads, D), dtype=x.dtype, device=x.device)
    _skiparse_ssp_pack(x, out, Bl // G, heads, T, H, W, D, s, group_size, _DTYPES[x.dtype], _stream())
    return out


def skiparse_ssp_unpack(recv: torch.Tensor, T: int, H: int, W: int, s: int, group_size: int, out: torch.Tensor | None = None):
    """The all-to-all receive buffer [group_size][G][G*b][base][heads][D] (chunk r came from rank r) -> the rank's shard
    [G*b][T*(H/s)*(W/s)][heads][D] in the other pattern's sparse layout."""
    gs, G, Bl, base, heads, D = recv.shape
    if gs != group_size or G * group_size != s * s or Bl % G or base * s * s * s * s != T * H * W:
        raise ValueError("receive-buffer shape does not match the grid and the group")
    if out is None:
        out = torch.empty((Bl, base * s * s, heads, D), dtype=recv.dtype, device=recv.device)
    _skiparse_ssp_unpack(recv, out, Bl // G, heads, T, H, W, D, s, group_size, _DTYPES[recv.dtype], _stream())
    return out


def dense_attn_fwd(q, k, v, T: int, H: int, W: int, scale: float = 0.0, out: torch.Tensor | None = None):
    """softmax(q k^T * scale) v over all T*H*W tokens for every (batch, head); bf16 in, bf16 out."""
    B, heads, D = _dims(q, T, H, W)
    if out is None:
        out = torch.empty_like(q)
    _dense_attn_fwd(q, k, v, out, B, heads, T, H, W, D, float(scale), _DTYPES[q.dtype], _stream())
    return out


def skiparse_workspace_bytes(B, heads, T, H, W, D, s, fused: bool) -> int:
    return int(lib().skiparse_workspace_bytes(B, heads, T, H, W, D, s, BF16, FUSED if fused else 0))


def skiparse_attn_fwd(q, k, v, T: int, H: int, W: int, s: int, pattern: str, scale: float = 0.0, fused: bool = True,
                      out: torch.Tensor | None = None, workspace: torch.Tensor | None = None, pad: bool = False):
    """Skiparse-2D attention, q/k/v/out in the original layout.  The unfused path needs a uint8 device workspace of
    skiparse_workspace_bytes() bytes; one is allocated with torch if none is passed.  pad=True selects the any-resolution
    mode (fused only): H and W arbitrary, end padding to multiples of s*s masked."""
    B, heads, D = _dims(q, T, H, W)
    if out is None:
        out = torch.empty_like(q)
    ws_bytes = 0
    if fused:
        workspace = None
    else:
        need = skiparse_workspace_bytes(B, heads, T, H, W, D, s, False)
        if workspace is None:
            workspace = torch.empty(max(need, 1), dtype=torch.uint8, device=q.device)
        ws_bytes = workspace.numel() * workspace.element_size()
    _skiparse_attn_fwd(q, k, v, out, B, heads, T, H, W, D, s, PATTERNS[pattern], float(scale), _DTYPES[q.dtype],
                       (FUSED if fused else 0) | (PAD if pad else 0), workspace, ws_bytes, _stream())
    return out


def skiparse_attn_fwd_sparse(q, k, v, T: int, H: int, W: int, s: int, pattern: str, out_layout: str = "other", scale: float = 0.0,
                             out: torch.Tensor | None = None):
    """Attention on tensors already in the sparse layout of `pattern` ([s*s*B][N/s^2][heads][D]); the output goes to the
    same layout ("same"), the other pattern's sparse layout ("other") or the original layout ("original")."""
    SB, Nsub, heads, D = q.shape
    B = SB // (s * s)
    if SB != B * s * s or Nsub * s * s != T * H * W:
        raise ValueError("sparse-layout shape does not match the grid")
    if out is None:
        shape = (B, T * H * W, heads, D) if out_layout == "original" else tuple(q.shape)
        out = torch.empty(shape, dtype=q.dtype, device=q.device)
    _skiparse_attn_fwd_sparse(q, k, v, out, B, heads, T, H, W, D, s, PATTERNS[pattern], OUT_LAYOUTS[out_layout], float(scale),
                              _DTYPES[q.dtype], _stream())
    return out


_INTS = (int,) * 9


@functools.lru_cache(maxsize=256)
def _bytes_of_ints(name: str, *sizes: int) -> int:
    return int(getattr(lib(), name)(*sizes))


def _bytes(name: str, *sizes) -> int:
    """A size that the library computes from (B, heads, T, H, W, D, s, pattern, flags).  Remembered for plain integers only: they are their
    own value, while a one-element tensor is looked up by identity and may change, and 8.0, which the call refuses, is found under 8."""
    if tuple(map(type, sizes)) == _INTS:
        return _bytes_of_ints(name, *sizes)
    return int(getattr(lib(), name)(*sizes))


def skiparse_lse_shape(B, heads, T, H, W, D, s, pattern: str, pad: bool = False):
    """Shape of the log-sum-exp tensor: [s*s*B][heads][positions per subsequence] (positions of the padded grid with pad=True)."""
    n = _bytes("skiparse_lse_bytes", B, heads, T, H, W, D, s, PATTERNS[pattern], PAD if pad else 0) // 4
    if n == 0:
        raise ValueError("grid does not fit the pattern (use pad=True for the any-resolution mode)")
    return (s * s * B, heads, n // (s * s * B * heads))


def skiparse_attn_fwd_lse(q, k, v, T: int, H: int, W: int, s: int, pattern: str, scale: float = 0.0,
                          out: torch.Tensor | None = None, lse: torch.Tensor | None = None, pad: bool = False):
    """Fused forward that also returns the log-sum-exp the backward pass needs: (out, lse), lse float32 in subsequence order."""
    B, heads, D = _dims(q, T, H, W)
    if out is None:
        out = torch.empty_like(q)
    if lse is None:
        lse = torch.empty(skiparse_lse_shape(B, heads, T, H, W, D, s, pattern, pad), dtype=torch.float32, device=q.device)
    _skiparse_attn_fwd_lse(q, k, v, out, lse, B, heads, T, H, W, D, s, PATTERNS[pattern], float(scale), _DTYPES[q.dtype], PAD if pad else 0,
                           _stream())
    return out, lse


def skiparse_bwd_workspace_bytes(B, heads, T, H, W, D, s, pattern: str, pad: bool = False) -> int:
    """Bytes that skiparse_attn_bwd cannot do without."""
    return _bytes("skiparse_bwd_workspace_bytes", B, heads, T, H, W, D, s, PATTERNS[pattern], PAD if pad else 0)


def skiparse_bwd_walk_workspace_bytes(B, heads, T, H, W, D, s, pattern: str, pad: bool = False) -> int:
    """Bytes with which skiparse_attn_bwd is fastest: more than the least for large problems at head_dim 128."""
    return _bytes("skiparse_bwd_walk_workspace_bytes", B, heads, T, H, W, D, s, PATTERNS[pattern], PAD if pad else 0)


def _bwd_workspace(device, *call) -> torch.Tensor:
    """For the fastest kernels (1.7 GB at 160 units of 20,160 positions), or where that is not to be had for the others (13 MB there)."""
    least, walk = skiparse_bwd_workspace_bytes(*call), skiparse_bwd_walk_workspace_bytes(*call)
    if walk > least:
        try:
            return torch.empty(walk, dtype=torch.uint8, device=device)
        except torch.cuda.OutOfMemoryError:
            pass
    return torch.empty(max(least, 1), dtype=torch.uint8, device=device)


def skiparse_attn_bwd(q, k, v, out, dout, lse, T: int, H: int, W: int, s: int, pattern: str, scale: float = 0.0,
                      dq=None, dk=None, dv=None, workspace: torch.Tensor | None = None, pad: bool = False):
    """Gradients (dq, dk, dv) of the Skiparse attention layer; out and lse come from skiparse_attn_fwd_lse (same pad flag).  A
    uint8 device workspace of skiparse_bwd_walk_workspace_bytes() bytes is allocated with torch if none is passed; a smaller one, down to
    skiparse_bwd_workspace_bytes(), selects kernels that need no more (slower on large problems at head_dim 128), as does a device that
    has no room for it.  The two round differently: pass a workspace where every call has to give the same bits."""
    B, heads, D = _dims(q, T, H, W)
    dq = torch.empty_like(q) if dq is None else dq
    dk = torch.empty_like(q) if dk is None else dk
    dv = torch.empty_like(q) if dv is None else dv
    if workspace is None:
        workspace = _bwd_workspace(q.device, B, heads, T, H, W, D, s, pattern, pad)
    _skiparse_attn_bwd(q, k, v, out, dout, lse, dq, dk, dv, B, heads, T, H, W, D, s, PATTERNS[pattern], float(scale), _DTYPES[q.dtype],
                       PAD if pad else 0, workspace, workspace.numel() * workspace.element_size(), _stream())
    return dq, dk, dv


def skiparse_attn_bwd_static(q, k, v, out, dout, lse, dq, dk, dv, T: int, H: int, W: int, s: int, pattern: str, scale: float = 0.0,
                             pad: bool = False):
    """skiparse_attn_bwd for callers that cannot allocate: the delta workspace is the library's static device array, and this
    wrapper allocates nothing either (dq, dk, dv must be passed).  Results are those of skiparse_attn_bwd with a workspace of
    skiparse_bwd_workspace_bytes() bytes; problems that need more than the array's size raise (code -4)."""
    B, heads, D = _dims(q, T, H, W)
    _skiparse_attn_bwd_static(q, k, v, out, dout, lse, dq, dk, dv, B, heads, T, H, W, D, s, PATTERNS[pattern], float(scale),
                              _DTYPES[q.dtype], PAD if pad else 0, _stream())
    return dq, dk, dv


def skiparse_quantize_fp8(x: torch.Tensor, T: int, H: int, W: int, s: int, pattern: str, pad: bool = False):
    """bf16 [B][N][heads][D] (original layout) -> (uint8 E4M3 codes [s*s*B][positions][heads][D] in the sparse layout,
    float32 scales [s*s*B][heads][ceil(positions/128)]).  positions = N/s^2, or with pad=True (any-resolution mode) the positions
    of the grid padded to multiples of s*s, with zero codes at the padding."""
    B, heads, D = _dims(x, T, H, W)
    if x.dtype != torch.bfloat16:
        raise ValueError("skiparse_quantize_fp8 takes bf16 input")
    nsub = skiparse_lse_shape(B, heads, T, H, W, D, s, pattern, pad)[2]
    x8 = torch.empty((s * s * B, nsub, heads, D), dtype=torch.uint8, device=x.device)
    scales = torch.empty((s * s * B, heads, (nsub + 127) // 128), dtype=torch.float32, device=x.device)
    _skiparse_quantize_fp8_ex(x, x8, scales, B, heads, T, H, W, D, s, PATTERNS[pattern], PAD if pad else 0, _stream())
    return x8, scales


def skiparse_attn_fwd_fp8(q8, k8, v8, sq, sk, sv, T: int, H: int, W: int, s: int, pattern: str, scale: float = 0.0,
                          out: torch.Tensor | None = None, pad: bool = False):
    """Attention on quantised sparse-layout tensors (from skiparse_quantize_fp8, same pad flag); bf16 output [B][N][heads][D] in the
    original layout."""
    SB, nsub, heads, D = q8.shape
    B = SB // (s * s)
    if SB != B * s * s or (not pad and nsub * s * s != T * H * W):
        raise ValueError("sparse-layout shape does not match the grid")
    if out is None:
        out = torch.empty((B, T * H * W, heads, D), dtype=torch.bfloat16, device=q8.device)
    _skiparse_attn_fwd_fp8_ex(q8, k8, v8, sq, sk, sv, out, B, heads, T, H, W, D, s, PATTERNS[pattern], float(scale), PAD if pad else 0,
                              _stream())
    return out
