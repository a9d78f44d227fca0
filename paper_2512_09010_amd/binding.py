"""ctypes binding over ``libluvc.so`` - same names as the C ABI in ``include/luvc.h``.

Argument marshalling only: every step of OIM and SPU runs in the HIP kernels.  PyTorch is used
for device memory (tensors own the buffers) and for the current stream handle.  There is no
CPU fallback: if the library is missing or cannot be loaded, importing callers get an error.

The calls that enqueue work go through ``_luvc_call`` (csrc/pycall.c) and ask for a workspace size only where
they allocate one: on small inputs a call is bound by what the host does before the launch (one 24x24 image through merge, score
and prune: 30 us of host time through ctypes, 14 like this).  Where ``_luvc_call`` is not built - it needs x86-64, gcc and the
Python headers - ctypes makes the same calls.
"""
from __future__ import annotations

import ctypes
import os
from itertools import chain
from typing import List, Optional, Sequence, Tuple

_HERE = os.path.dirname(os.path.abspath(__file__))
# LUVC_HOST_SANITIZE=1 loads the build whose host code carries the sanitizers (see build.py)
LIB_PATH = os.path.join(_HERE, "libluvc_san.so" if os.environ.get("LUVC_HOST_SANITIZE", "") not in ("", "0") else "libluvc.so")

LUVC_OK, LUVC_ERR_INVALID_ARG, LUVC_ERR_UNSUPPORTED, LUVC_ERR_WORKSPACE, LUVC_ERR_HIP = range(5)
LUVC_F32, LUVC_BF16 = 0, 1

EXPORTS = ("luvc_version", "luvc_last_error", "luvc_oim_plan", "luvc_oim_workspace_bytes", "luvc_oim_merge",
           "luvc_oim_wide_workspace_bytes", "luvc_oim_merge_wide",
           "luvc_oim_keyed_workspace_bytes", "luvc_oim_merge_keyed", "luvc_value_enhance", "luvc_spu_workspace_bytes", "luvc_spu_score", "luvc_spu_score_static", "luvc_keep_count", "luvc_spu_prune",
           "luvc_spu_cascade_keeps", "luvc_spu_stage",
           "luvc_oim_plan_anyres", "luvc_oim_ragged_workspace_bytes", "luvc_oim_merge_ragged",
           "luvc_spu_ragged_workspace_bytes", "luvc_spu_stage_ragged",
           "luvc_profile_start", "luvc_profile_stop", "luvc_profile_kernel", "luvc_selftest_fdot2", "luvc_selftest_screen_tile",
           "luvc_selftest_screen_bound")


class LuvcPass(ctypes.Structure):
    _fields_ = [("axis", ctypes.c_int32), ("m", ctypes.c_int32)]


class LuvcError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"libluvc status {status}: {text}")
        self.status = status


_lib = None


def lib() -> ctypes.CDLL:
    """Load libluvc.so (built beforehand by ``paper_2512_09010_amd.build``); raises if it is absent."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(f"{LIB_PATH} is not built; run `python -m paper_2512_09010_amd.build` "
                                "(there is no fallback implementation)")
    L = ctypes.CDLL(LIB_PATH)
    i, i64, vp, sz = ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t
    pp = ctypes.POINTER(LuvcPass)
    L.luvc_version.restype = ctypes.c_char_p
    L.luvc_last_error.restype = ctypes.c_char_p
    L.luvc_oim_plan.argtypes = [i, i, i64, pp, i, ctypes.POINTER(i)]
    L.luvc_oim_plan.restype = i
    L.luvc_oim_workspace_bytes.argtypes = [i, i, i, i, i, pp, i]
    L.luvc_oim_workspace_bytes.restype = sz
    L.luvc_oim_merge.argtypes = [vp, vp, i, i, i, i, i, pp, i, i64, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_oim_merge.restype = i
    L.luvc_oim_wide_workspace_bytes.argtypes = [i, i, i, i, i, pp, i, i]
    L.luvc_oim_wide_workspace_bytes.restype = sz
    L.luvc_oim_merge_wide.argtypes = [vp, vp, i, i, i, i, i, pp, i, i, i64, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_oim_merge_wide.restype = i
    L.luvc_oim_keyed_workspace_bytes.argtypes = [i, i, i, i, i, i, pp, i, i]
    L.luvc_oim_keyed_workspace_bytes.restype = sz
    L.luvc_oim_merge_keyed.argtypes = [vp, vp, vp, i, i, i, i, i, i, pp, i, i, i64, vp, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_oim_merge_keyed.restype = i
    L.luvc_value_enhance.argtypes = [vp, vp, i64, i, i64, i, vp, i64, vp]
    L.luvc_value_enhance.restype = i
    L.luvc_spu_workspace_bytes.argtypes = [i, i, i, i, i]
    L.luvc_spu_workspace_bytes.restype = sz
    L.luvc_spu_score.argtypes = [vp, i, i, i, i64, i, i, i, vp, vp, sz, vp]
    L.luvc_spu_score.restype = i
    L.luvc_spu_score_static.argtypes = [vp, i, i, i, i64, i, i, i, vp, vp]
    L.luvc_spu_score_static.restype = i
    L.luvc_keep_count.argtypes = [i, ctypes.c_double]
    L.luvc_keep_count.restype = i
    L.luvc_spu_prune.argtypes = [vp, vp, i, i, i, i64, i, i, vp, vp, vp, sz, vp]
    L.luvc_spu_prune.restype = i
    L.luvc_spu_cascade_keeps.argtypes = [i, ctypes.c_double, i, i, ctypes.POINTER(ctypes.c_int)]
    L.luvc_spu_cascade_keeps.restype = i
    L.luvc_spu_stage.argtypes = [vp, i, i, i, i64, i, i, i, i, vp, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_spu_stage.restype = i
    ip = ctypes.POINTER(ctypes.c_int32)
    L.luvc_oim_plan_anyres.argtypes = [i, i, i64, pp, i, ctypes.POINTER(ctypes.c_int)]
    L.luvc_oim_plan_anyres.restype = i
    L.luvc_oim_ragged_workspace_bytes.argtypes = [i, ip, ip, i, i, pp, ip]
    L.luvc_oim_ragged_workspace_bytes.restype = sz
    L.luvc_oim_merge_ragged.argtypes = [vp, vp, i, ip, ip, i, i, pp, ip, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_oim_merge_ragged.restype = i
    L.luvc_spu_ragged_workspace_bytes.argtypes = [i, ip, i, i, ip]
    L.luvc_spu_ragged_workspace_bytes.restype = sz
    L.luvc_spu_stage_ragged.argtypes = [vp, i, ip, i, i64, i, ip, i, ip, vp, vp, vp, vp, vp, vp, sz, vp]
    L.luvc_spu_stage_ragged.restype = i
    L.luvc_profile_start.argtypes = [ctypes.POINTER(vp), i]
    L.luvc_profile_start.restype = i
    L.luvc_profile_stop.argtypes = []
    L.luvc_profile_stop.restype = i
    L.luvc_profile_kernel.argtypes = [i]
    L.luvc_profile_kernel.restype = ctypes.c_char_p
    L.luvc_selftest_fdot2.argtypes = [vp, vp, i, i, vp, vp]
    L.luvc_selftest_fdot2.restype = i
    L.luvc_selftest_screen_tile.argtypes = [vp, vp, i, i, vp, vp]
    L.luvc_selftest_screen_tile.restype = i
    L.luvc_selftest_screen_bound.argtypes = [i, i, ctypes.POINTER(i), ctypes.POINTER(ctypes.c_float)]
    L.luvc_selftest_screen_bound.restype = i
    _lib = L
    return L


class _Native:
    """What a call needs at hand: torch, the caller, the addresses of the entry points."""

    def __init__(self):
        import torch
        L = lib()
        try:
            from ._luvc_call import call
        except ImportError:                             # hosts it is not built for: the same calls through ctypes
            call = None
        self.torch, self.call = torch, call or (lambda entry, *args: entry(*args))
        self.code = {torch.float32: LUVC_F32, torch.bfloat16: LUVC_BF16}
        self.i32, self.f32 = torch.int32, torch.float32
        self.raw_stream, self.device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice
        for name in ("luvc_oim_merge", "luvc_oim_merge_wide", "luvc_oim_merge_keyed", "luvc_value_enhance", "luvc_spu_score", "luvc_spu_score_static",
                     "luvc_spu_prune", "luvc_spu_stage", "luvc_oim_merge_ragged", "luvc_spu_stage_ragged"):
            f = getattr(L, name)
            entry = ctypes.cast(f, ctypes.c_void_p).value
            if call is None:                            # host arrays are handed over as addresses here too
                entry = ctypes.CFUNCTYPE(f.restype, *(ctypes.c_void_p if issubclass(t, ctypes._Pointer) else t for t in f.argtypes))(entry)
            setattr(self, name, entry)

    def stream(self, stream) -> int:
        return self.raw_stream(self.device()) if stream is None else int(stream.cuda_stream)


_native_state = None


def _native() -> _Native:
    global _native_state
    if _native_state is None:
        _native_state = _Native()
    return _native_state


def last_error() -> str:
    return lib().luvc_last_error().decode()


def _check(status: int):
    if status != LUVC_OK:
        raise LuvcError(status, last_error())


def _passes(passes: Sequence[Tuple[int, int]]):
    arr = (LuvcPass * max(1, len(passes)))()
    for k, (axis, m) in enumerate(passes):
        arr[k].axis, arr[k].m = int(axis), int(m)
    return arr


class _Bounded(dict):
    """Marshalled argument lists by what they were made from; emptied when full."""

    def keep(self, key, value, most=128):
        if len(self) >= most:
            self.clear()
        self[key] = value
        return value


def _ints(*lists) -> bool:
    """Only tuples of plain ints become a key: an entry that may be changed in place (a 0-d tensor hashes by identity) would
    be found again with another value.  Looking up needs no such care: what equals a tuple of ints holds these values now."""
    return set(map(type, lists)) <= {tuple} and set(map(type, chain.from_iterable(lists))) <= {int}


_schedules = _Bounded()


def _schedule(passes):
    """(ctypes array, its address, length) of a schedule."""
    try:
        key = tuple(passes)
        hit = _schedules.get(key)
    except TypeError:                                   # entries that do not hash
        key, hit = None, None
    if hit is None:
        arr = _passes(passes)
        hit = (arr, ctypes.addressof(arr), len(passes))
        if key is not None and _ints(*key):
            _schedules.keep(key, hit)
    return hit


def _dtype_code(t) -> int:
    code = _native().code.get(t.dtype)
    if code is None:
        raise TypeError(f"unsupported dtype {t.dtype}")
    return code


def _ptr(t) -> Optional[int]:
    return None if t is None else t.data_ptr()


def luvc_version() -> str:
    return lib().luvc_version().decode()


def luvc_keep_count(N: int, keep_ratio: float) -> int:
    return lib().luvc_keep_count(int(N), float(keep_ratio))


def luvc_oim_plan(H: int, W: int, target_tokens: int, max_passes: int = 16) -> List[Tuple[int, int]]:
    arr = (LuvcPass * max_passes)()
    n = ctypes.c_int(0)
    _check(lib().luvc_oim_plan(H, W, int(target_tokens), arr, max_passes, ctypes.byref(n)))
    return [(arr[k].axis, arr[k].m) for k in range(n.value)]


def luvc_oim_workspace_bytes(B, H, W, D, dtype_code, passes) -> int:
    return lib().luvc_oim_workspace_bytes(B, H, W, D, dtype_code, _passes(passes), len(passes))


def out_grid(H: int, W: int, passes) -> Tuple[int, int]:
    for axis, m in passes:                              # not in place: H and W may be the caller's 0-d tensors
        if axis == 1:
            W = W - m
        else:
            H = H - m
    return H, W


def _merge_outputs(t, x, Ho, Wo, want_maps):
    B, H, W, D = x.shape
    Ho, Wo = max(Ho, 0), max(Wo, 0)
    i32 = dict(dtype=t.int32, device=x.device)
    return dict(x=t.empty((B, Ho, Wo, D), dtype=x.dtype, device=x.device), sizes=t.empty((B, Ho, Wo), **i32),
                merged_map=t.empty((B, H * W), **i32) if want_maps else None, kept_map=t.empty((B, Ho * Wo), **i32) if want_maps else None)


def _map_ptrs(out):
    m, k = out.get("merged_map"), out.get("kept_map")
    return None if m is None else m.data_ptr(), None if k is None else k.data_ptr()


def luvc_oim_merge(x, passes, sizes=None, target_tokens: int = 0, want_maps: bool = True, workspace=None, stream=None,
                   out=None):
    """x: CUDA tensor [B,H,W,D] (fp32 or bf16, contiguous).  Returns dict(x, sizes, merged_map, kept_map)."""
    nat = _native()
    assert x.is_cuda and x.is_contiguous() and x.dim() == 4
    B, H, W, D = x.shape
    code = _dtype_code(x)
    arr, addr, n = _schedule(passes)
    if workspace is None:
        need = lib().luvc_oim_workspace_bytes(B, H, W, D, code, arr, n)
        workspace = nat.torch.empty(max(need, 256), dtype=nat.torch.uint8, device=x.device)
    if out is None:
        out = _merge_outputs(nat.torch, x, *out_grid(H, W, passes), want_maps)
    if sizes is not None:
        assert sizes.is_cuda and sizes.dtype == nat.i32 and sizes.is_contiguous() and sizes.numel() == B * H * W
        sizes = sizes.data_ptr()
    merged, kept = _map_ptrs(out)
    _check(nat.call(nat.luvc_oim_merge, x.data_ptr(), sizes, B, H, W, D, code, addr, n, int(target_tokens),
                    out["x"].data_ptr(), out["sizes"].data_ptr(), merged, kept, workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return out


def luvc_oim_wide_workspace_bytes(B, H, W, D, dtype_code, passes, radius) -> int:
    return lib().luvc_oim_wide_workspace_bytes(B, H, W, D, dtype_code, _passes(passes), len(passes), int(radius))


def luvc_oim_merge_wide(x, passes, radius: int, sizes=None, target_tokens: int = 0, want_maps: bool = True, workspace=None,
                        stream=None, out=None):
    """As luvc_oim_merge with candidates within `radius` (0 = the whole line).  Returns dict(x, sizes, merged_map, kept_map)."""
    nat = _native()
    assert x.is_cuda and x.is_contiguous() and x.dim() == 4
    B, H, W, D = x.shape
    code = _dtype_code(x)
    arr, addr, n = _schedule(passes)
    if workspace is None:
        need = lib().luvc_oim_wide_workspace_bytes(B, H, W, D, code, arr, n, int(radius))
        workspace = nat.torch.empty(max(need, 256), dtype=nat.torch.uint8, device=x.device)
    if out is None:
        out = _merge_outputs(nat.torch, x, *out_grid(H, W, passes), want_maps)
    if sizes is not None:
        assert sizes.is_cuda and sizes.dtype == nat.i32 and sizes.is_contiguous() and sizes.numel() == B * H * W
        sizes = sizes.data_ptr()
    merged, kept = _map_ptrs(out)
    _check(nat.call(nat.luvc_oim_merge_wide, x.data_ptr(), sizes, B, H, W, D, code, addr, n, int(radius), int(target_tokens),
                    out["x"].data_ptr(), out["sizes"].data_ptr(), merged, kept, workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return out


def luvc_oim_keyed_workspace_bytes(B, H, W, D, Dm, dtype_code, passes, radius) -> int:
    return lib().luvc_oim_keyed_workspace_bytes(B, H, W, D, Dm, dtype_code, _passes(passes), len(passes), int(radius))


def luvc_oim_merge_keyed(x, metric, passes, radius: int = 1, sizes=None, target_tokens: int = 0, want_maps: bool = True,
                         want_metric: bool = True, workspace=None, stream=None, out=None):
    """Decisions on metric [B,H,W,Dm], merge applied to x [B,H,W,D].  Returns dict(x, metric, sizes, merged_map, kept_map)."""
    nat = _native()
    assert x.is_cuda and x.is_contiguous() and x.dim() == 4 and metric.is_cuda and metric.is_contiguous() and metric.dim() == 4
    assert metric.shape[:3] == x.shape[:3] and metric.dtype == x.dtype
    B, H, W, D = x.shape
    Dm = metric.shape[3]
    code = _dtype_code(x)
    arr, addr, n = _schedule(passes)
    if workspace is None:
        need = lib().luvc_oim_keyed_workspace_bytes(B, H, W, D, Dm, code, arr, n, int(radius))
        workspace = nat.torch.empty(max(need, 256), dtype=nat.torch.uint8, device=x.device)
    if out is None:
        Ho, Wo = out_grid(H, W, passes)
        out = _merge_outputs(nat.torch, x, Ho, Wo, want_maps)
        out["metric"] = nat.torch.empty((B, max(Ho, 0), max(Wo, 0), Dm), dtype=x.dtype, device=x.device) if want_metric else None
    if sizes is not None:
        assert sizes.is_cuda and sizes.dtype == nat.i32 and sizes.is_contiguous() and sizes.numel() == B * H * W
        sizes = sizes.data_ptr()
    merged, kept = _map_ptrs(out)
    _check(nat.call(nat.luvc_oim_merge_keyed, x.data_ptr(), metric.data_ptr(), sizes, B, H, W, D, Dm, code, addr, n, int(radius),
                    int(target_tokens), out["x"].data_ptr(), _ptr(out.get("metric")), out["sizes"].data_ptr(), merged, kept,
                    workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return out


def luvc_value_enhance(v, sizes, stream=None, out=None):
    """v: CUDA tensor [..., D] (last dim contiguous, rows evenly strided), sizes int32 [...]: returns v + log(sizes)."""
    nat = _native()
    assert v.is_cuda and v.stride(-1) == 1 and sizes.is_cuda and sizes.dtype == nat.i32 and sizes.is_contiguous()
    D = v.shape[-1]
    rows = sizes.numel()
    assert v.numel() == rows * D and v.is_contiguous()
    if out is None:
        out = nat.torch.empty_like(v)
    _check(nat.call(nat.luvc_value_enhance, v.data_ptr(), sizes.data_ptr(), rows, D, D, _dtype_code(v), out.data_ptr(), D, nat.stream(stream)))
    return out


def luvc_spu_workspace_bytes(B, N, D, dtype_code, sigma) -> int:
    return lib().luvc_spu_workspace_bytes(B, N, D, dtype_code, sigma)


def luvc_spu_score(x, sigma: int, use_hamming: bool = True, workspace=None, stream=None, out=None):
    """x: CUDA tensor [B,N,D] (last dim contiguous; token stride may exceed D).  Returns scores [B,N] fp32."""
    nat = _native()
    B, N, D = x.shape
    sb, sn, sd = x.stride()
    assert x.is_cuda and sd == 1 and sb == N * sn
    code = _dtype_code(x)
    if workspace is None:
        need = lib().luvc_spu_workspace_bytes(B, N, D, code, int(sigma))
        workspace = nat.torch.empty(max(need, 256), dtype=nat.torch.uint8, device=x.device)
    if out is None:
        out = nat.torch.empty((B, N), dtype=nat.f32, device=x.device)
    _check(nat.call(nat.luvc_spu_score, x.data_ptr(), B, N, D, sn, code, int(sigma), int(bool(use_hamming)), out.data_ptr(),
                    workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return out


SPU_STATIC_SCRATCH_BYTES = 8 << 20


def luvc_spu_score_static(x, sigma: int, use_hamming: bool = True, stream=None, out=None):
    """luvc_spu_score on the library's static scratch (no workspace; pass `out` to keep the call free of allocations)."""
    nat = _native()
    assert x.is_cuda and x.dim() == 3 and x.stride(2) == 1 and x.stride(0) == x.shape[1] * x.stride(1)
    B, N, D = x.shape
    if out is None:
        out = nat.torch.empty((B, N), dtype=nat.f32, device=x.device)
    _check(nat.call(nat.luvc_spu_score_static, x.data_ptr(), B, N, D, x.stride(1), _dtype_code(x), int(sigma), int(bool(use_hamming)),
                    out.data_ptr(), nat.stream(stream)))
    return out


def luvc_spu_prune(x, scores, n_keep: int, gather: bool = True, stream=None, out=None):
    """Returns dict(kept_idx [B,n_keep] int32 ascending, x [B,n_keep,D] or None)."""
    nat = _native()
    assert scores.is_cuda and scores.dtype == nat.f32 and scores.is_contiguous() and scores.dim() == 2
    B, N = scores.shape
    D, stride, code, xp = 1, 1, LUVC_F32, None
    if x is not None:
        assert x.is_cuda and x.dim() == 3 and x.stride(2) == 1 and x.shape[:2] == scores.shape
        D, stride, code, xp = x.shape[2], x.stride(1), _dtype_code(x), x.data_ptr()
    if out is None:
        out = dict(kept_idx=nat.torch.empty((B, max(n_keep, 0)), dtype=nat.i32, device=scores.device),
                   x=nat.torch.empty((B, max(n_keep, 0), D), dtype=x.dtype, device=x.device) if (gather and x is not None) else None)
    _check(nat.call(nat.luvc_spu_prune, xp, scores.data_ptr(), B, N, D, stride, code, int(n_keep), out["kept_idx"].data_ptr(),
                    _ptr(out.get("x")), None, 0, nat.stream(stream)))
    return out


def luvc_spu_cascade_keeps(N0: int, keep_ratio: float, n_stages: int, eliminate: bool = True):
    """Keep counts of the stages of a cascade: one keep ratio stage after stage, 0 at the end when eliminate."""
    keeps = (ctypes.c_int * max(int(n_stages), 1))()
    n = lib().luvc_spu_cascade_keeps(int(N0), float(keep_ratio), int(n_stages), int(bool(eliminate)), keeps)
    if n != n_stages or n_stages < 1:
        raise LuvcError(LUVC_ERR_INVALID_ARG, "luvc_spu_cascade_keeps rejected its arguments")
    return [int(k) for k in keeps[:n]]


def luvc_spu_stage(x, sigma: int, n_keep: int, use_hamming: bool = True, origin=None, gather: bool = True,
                   workspace=None, stream=None, out=None):
    """One cascade stage on x [B,N,D].  Returns dict(scores [B,N] fp32, kept_idx, origin [B,n_keep] int32,
    x [B,n_keep,D] or None); with n_keep = 0 nothing is launched and the tensors are empty."""
    nat = _native()
    B, N, D = x.shape
    sb, sn, sd = x.stride()
    assert x.is_cuda and sd == 1 and sb == N * sn
    code = _dtype_code(x)
    if origin is not None:
        assert origin.is_cuda and origin.dtype == nat.i32 and origin.is_contiguous() and tuple(origin.shape) == (B, N)
        origin = origin.data_ptr()
    k = max(int(n_keep), 0)
    if workspace is None:
        need = lib().luvc_spu_workspace_bytes(B, N, D, code, int(sigma)) if k else 0
        workspace = nat.torch.empty(max(need, 256), dtype=nat.torch.uint8, device=x.device)
    if out is None:
        out = dict(scores=nat.torch.empty((B, N), dtype=nat.f32, device=x.device),
                   kept_idx=nat.torch.empty((B, k), dtype=nat.i32, device=x.device),
                   origin=nat.torch.empty((B, k), dtype=nat.i32, device=x.device),
                   x=nat.torch.empty((B, k, D), dtype=x.dtype, device=x.device) if gather else None)
    _check(nat.call(nat.luvc_spu_stage, x.data_ptr(), B, N, D, sn, code, int(sigma), int(bool(use_hamming)), int(n_keep),
                    origin, out["scores"].data_ptr(), out["kept_idx"].data_ptr(), out["origin"].data_ptr(),
                    _ptr(out.get("x")), workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return out


def _i32(values):
    return (ctypes.c_int32 * max(1, len(values)))(*[int(v) for v in values])


def luvc_oim_plan_anyres(H: int, W: int, max_tokens: int, max_passes: int = 16) -> List[Tuple[int, int]]:
    arr = (LuvcPass * max_passes)()
    n = ctypes.c_int(0)
    _check(lib().luvc_oim_plan_anyres(H, W, int(max_tokens), arr, max_passes, ctypes.byref(n)))
    return [(arr[k].axis, arr[k].m) for k in range(n.value)]


_ragged_merges, _ragged_stages = _Bounded(), _Bounded()


class _RaggedMerge:
    """The host arrays of a ragged merge and what follows from them."""

    def __init__(self, shapes, schedules, D, code):
        flat = [p for sch in schedules for p in sch]
        self.H, self.W = _i32([h for h, _ in shapes]), _i32([w for _, w in shapes])
        self.passes, self.n_passes = _passes(flat), _i32([len(sch) for sch in schedules])
        self.n = len(shapes)
        self.out_shapes = [out_grid(h, w, sch) for (h, w), sch in zip(shapes, schedules)]
        self.tokens_in = sum(h * w for h, w in shapes)
        self.tokens_out = sum(max(h, 0) * max(w, 0) for h, w in self.out_shapes)
        self.need = lib().luvc_oim_ragged_workspace_bytes(self.n, self.H, self.W, D, code, self.passes, self.n_passes)
        self.addr = [ctypes.addressof(a) for a in (self.H, self.W, self.passes, self.n_passes)]


def _merge_plan(shapes, schedules, D, code) -> _RaggedMerge:
    try:
        key = (D, code, tuple(shapes), tuple(map(tuple, schedules)))
        plan = _ragged_merges.get(key)
    except TypeError:                                   # entries that do not hash
        key, plan = None, None
    if plan is None:
        plan = _RaggedMerge(shapes, schedules, D, code)
        if key is not None and _ints(*key[2], *chain.from_iterable(key[3])):
            _ragged_merges.keep(key, plan)
    return plan


def luvc_oim_merge_ragged(x, shapes, schedules, sizes=None, want_maps: bool = True, workspace=None, stream=None):
    """x: CUDA tensor [sum H_i*W_i, D], image after image; shapes [(H_i, W_i)]; schedules: one pass list per image.
    Returns dict(x [sum H'_i*W'_i, D], sizes, merged_map, kept_map, out_shapes)."""
    nat = _native()
    torch = nat.torch
    assert x.is_cuda and x.is_contiguous() and x.dim() == 2 and len(shapes) == len(schedules)
    T, D = x.shape
    code = _dtype_code(x)
    plan = _merge_plan(shapes, schedules, D, code)
    assert T == plan.tokens_in
    To = plan.tokens_out
    if workspace is None:
        workspace = torch.empty(max(plan.need, 256), dtype=torch.uint8, device=x.device)
    if sizes is not None:
        assert sizes.is_cuda and sizes.dtype == nat.i32 and sizes.is_contiguous() and sizes.numel() == T
        sizes = sizes.data_ptr()
    xo = torch.empty((To, D), dtype=x.dtype, device=x.device)
    so = torch.empty((To,), dtype=nat.i32, device=x.device)
    merged = torch.empty((T,), dtype=nat.i32, device=x.device) if want_maps else None
    kept = torch.empty((To,), dtype=nat.i32, device=x.device) if want_maps else None
    H, W, passes, n_passes = plan.addr
    _check(nat.call(nat.luvc_oim_merge_ragged, x.data_ptr(), sizes, plan.n, H, W, D, code, passes, n_passes, xo.data_ptr(), so.data_ptr(),
                    _ptr(merged), _ptr(kept), workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return dict(x=xo, sizes=so, merged_map=merged, kept_map=kept, out_shapes=list(plan.out_shapes))


class _RaggedStage:
    """The host arrays of a ragged stage and what follows from them."""

    def __init__(self, lengths, sigmas, keeps, D, code):
        self.N, self.sigma = _i32(lengths), _i32(sigmas)
        self.keep = _i32(keeps) if keeps is not None else None
        self.n = len(lengths)
        self.tokens = sum(lengths)
        self.kept = sum(max(int(k), 0) for k in keeps) if keeps is not None else 0
        self.need = lib().luvc_spu_ragged_workspace_bytes(self.n, self.N, D, code, self.sigma)
        self.addr = [None if a is None else ctypes.addressof(a) for a in (self.N, self.sigma, self.keep)]


def _stage_plan(lengths, sigmas, keeps, D, code) -> _RaggedStage:
    try:
        key = (D, code, tuple(lengths), tuple(sigmas), None if keeps is None else tuple(keeps))
        plan = _ragged_stages.get(key)
    except TypeError:
        key, plan = None, None
    if plan is None:
        plan = _RaggedStage(lengths, sigmas, keeps, D, code)
        if key is not None and _ints(*key[2:4], key[4] or ()):
            _ragged_stages.keep(key, plan)
    return plan


def luvc_spu_stage_ragged(x, lengths, sigmas, keeps=None, use_hamming: bool = True, origin=None, gather: bool = True,
                          workspace=None, stream=None):
    """x: CUDA tensor [sum N_i, D] (rows evenly strided), sample after sample; lengths, sigmas, keeps: per sample.
    Returns dict(scores [sum N_i] fp32, kept_idx, origin [sum keep_i] int32, x [sum keep_i, D] or None)."""
    nat = _native()
    torch = nat.torch
    assert x.is_cuda and x.dim() == 2 and x.stride(1) == 1 and len(lengths) == len(sigmas)
    T, D = x.shape
    code = _dtype_code(x)
    plan = _stage_plan(lengths, sigmas, keeps, D, code)
    assert T == plan.tokens
    K = plan.kept
    if origin is not None:
        assert origin.is_cuda and origin.dtype == nat.i32 and origin.is_contiguous() and origin.numel() == T
        origin = origin.data_ptr()
    if workspace is None:
        workspace = torch.empty(max(plan.need, 256), dtype=torch.uint8, device=x.device)
    scores = torch.empty((T,), dtype=nat.f32, device=x.device)
    kept_idx, kept_origin = torch.empty((K,), dtype=nat.i32, device=x.device), torch.empty((K,), dtype=nat.i32, device=x.device)
    xo = torch.empty((K, D), dtype=x.dtype, device=x.device) if (gather and keeps is not None) else None
    # a tensor without elements has no address: hand the library one it will not touch
    ki = kept_idx.data_ptr() if K else scores.data_ptr()
    og = kept_origin.data_ptr() if K else scores.data_ptr()
    N, sigma, keep = plan.addr
    _check(nat.call(nat.luvc_spu_stage_ragged, x.data_ptr(), plan.n, N, D, x.stride(0), code, sigma, int(bool(use_hamming)), keep,
                    origin, scores.data_ptr(), ki, og, _ptr(xo) if K else None, workspace.data_ptr(), workspace.numel(), nat.stream(stream)))
    return dict(scores=scores, kept_idx=kept_idx, origin=kept_origin, x=xo)


class LaunchProfile:
    """Durations of the kernels libluvc launches between start() and stop(), from HIP events recorded on
    the launch stream (luvc_profile_start / luvc_profile_stop).  Only marshals: the events come from the
    HIP runtime, the recording is done by the library."""

    def __init__(self, max_launches: int):
        self._hip = ctypes.CDLL("libamdhip64.so")
        self._hip.hipEventCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
        self._hip.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]
        self._hip.hipEventSynchronize.argtypes = [ctypes.c_void_p]
        self._hip.hipEventDestroy.argtypes = [ctypes.c_void_p]
        self.n = 2 * int(max_launches)
        self.events = (ctypes.c_void_p * self.n)()
        for k in range(self.n):
            e = ctypes.c_void_p()
            if self._hip.hipEventCreate(ctypes.byref(e)) != 0:
                raise RuntimeError("hipEventCreate failed")
            self.events[k] = e
        self.count = 0

    def start(self):
        _check(lib().luvc_profile_start(self.events, self.n))

    def stop(self) -> int:
        self.count = lib().luvc_profile_stop()
        return self.count

    def results(self):
        """[(kernel name, milliseconds)] in launch order; call after the stream has been synchronised."""
        out = []
        for k in range(self.count):
            ms = ctypes.c_float(0)
            self._hip.hipEventSynchronize(self.events[2 * k + 1])
            if self._hip.hipEventElapsedTime(ctypes.byref(ms), self.events[2 * k], self.events[2 * k + 1]) != 0:
                raise RuntimeError("hipEventElapsedTime failed")
            out.append((lib().luvc_profile_kernel(k).decode(), float(ms.value)))
        return out

    def close(self):
        for k in range(self.n):
            if self.events[k]:
                self._hip.hipEventDestroy(self.events[k])
                self.events[k] = None


def luvc_selftest_fdot2(x, y, stream=None):
    """x, y [rows, 2 * words] bf16 -> [rows] fp32: the packed bf16 dot product instruction chained over a row."""
    import torch
    assert x.is_cuda and x.dtype == torch.bfloat16 and x.shape == y.shape and x.dim() == 2 and x.shape[1] % 2 == 0
    assert x.is_contiguous() and y.is_contiguous()
    out = torch.empty((x.shape[0],), dtype=torch.float32, device=x.device)
    _check(lib().luvc_selftest_fdot2(_ptr(x), _ptr(y), x.shape[0], x.shape[1] // 2, _ptr(out), _native().stream(stream)))
    return out


def luvc_selftest_screen_tile(a, c, stream=None):
    """a, c [32, D] (fp32 or bf16) -> [32, 32] fp32: the screening tile of the wide matching, <a_i, c_j> on the matrix cores."""
    import torch
    assert a.is_cuda and a.shape == c.shape and a.dim() == 2 and a.shape[0] == 32 and a.dtype == c.dtype
    assert a.is_contiguous() and c.is_contiguous()
    out = torch.empty((32, 32), dtype=torch.float32, device=a.device)
    _check(lib().luvc_selftest_screen_tile(_ptr(a), _ptr(c), a.shape[1], _dtype_code(a), _ptr(out), _native().stream(stream)))
    return out


def luvc_selftest_screen_bound(D, dtype):
    """-> (channels, eps): the most channels a wavefront of the wide matching's screening contracts for rows of D, and what a screened cosine is taken to be within."""
    c, eps = ctypes.c_int(), ctypes.c_float()
    _check(lib().luvc_selftest_screen_bound(D, dtype, ctypes.byref(c), ctypes.byref(eps)))
    return c.value, eps.value
