"""Thin ctypes binding over liblagkv.so (the C ABI declared in include/lagkv.h).

Argument marshalling only: every step of the pass runs in the HIP kernels.
Functions carry the C names (`plan`, `workspace_bytes`, `score`, `select`,
`compress`, `append_and_compress`, `launch_hint`, ...).  torch is used for device memory
and the current HIP stream; there is no CPU fallback: if the library is
missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes as C
import functools
import importlib
import os
import warnings
from dataclasses import dataclass
from operator import index
from typing import Optional, Tuple

import torch

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "liblagkv.so")
_lib = None
_native = None  # csrc/binding.cpp, once the library is loaded (None where it is not built: the ctypes calls below do the same)

OK, EINVAL, ESHAPE, EDTYPE, ECAPACITY, EWORKSPACE, EHIP = range(7)
F32, BF16, F16 = 0, 1, 2
SCORE_LAG, SCORE_LOCAL, SCORE_L2 = 0, 1, 2
PATH_AUTO, PATH_FUSED, PATH_STAGED, PATH_RESIDENT = 0, 1, 2, 3
ORDER_LINEAR, ORDER_EVEN_ODD, ORDER_XCD, ORDER_BITREV = 0, 1, 2, 3
SELECT_AUTO, SELECT_WAVE, SELECT_GROUP = 0, 1, 2

EXPORTS = ("lagkv_plan", "lagkv_keep_for_compression", "lagkv_workspace_bytes", "lagkv_score",
           "lagkv_select", "lagkv_compress", "lagkv_compress_static", "lagkv_cache_after_compress",
           "lagkv_prefill_rows",
           "lagkv_append_and_compress", "lagkv_prefill", "lagkv_launch_hint", "lagkv_launch_hint_ex", "lagkv_path_for",
           "lagkv_kernel_for", "lagkv_strerror",
           "lagkv_version")


class LagKVError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {strerror(status)} (status {status})")


class Params(C.Structure):
    _fields_ = [("B", C.c_int32), ("H", C.c_int32), ("D", C.c_int32),
                ("S", C.c_int32), ("L", C.c_int32),
                ("r", C.c_double),
                ("dtype", C.c_int32), ("variant", C.c_int32), ("std_ddof", C.c_int32),
                ("launch", C.c_int32),
                ("stride_b", C.c_int64), ("stride_h", C.c_int64), ("stride_t", C.c_int64)]


class PlanT(C.Structure):
    _fields_ = [("n_chunks", C.c_int64), ("n_scored", C.c_int64), ("rem", C.c_int64),
                ("k", C.c_int64), ("T_out", C.c_int64)]


class CacheT(C.Structure):
    _fields_ = [("K", C.c_void_p), ("V", C.c_void_p), ("pos", C.c_void_p),
                ("capacity", C.c_int64), ("n_static", C.c_int64), ("n_tail", C.c_int64),
                ("n_seen", C.c_int64)]


def lib_path() -> str:
    return _LIB_PATH


def load():
    """Load liblagkv.so (built by paper_2504_04704_amd.build / __graft_entry__.build)."""
    global _lib, _native
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} is missing: run `python -c 'import __graft_entry__ as g; "
                          f"g.build()'` (hipcc, gfx950) first; there is no fallback path")
    lib = C.CDLL(_LIB_PATH)
    vp, i64, sz = C.c_void_p, C.c_int64, C.c_size_t
    lib.lagkv_plan.argtypes = [C.POINTER(Params), i64, i64, C.POINTER(PlanT)]
    lib.lagkv_plan.restype = C.c_int
    lib.lagkv_keep_for_compression.argtypes = [i64, C.c_int32, C.c_int32, C.c_double,
                                               C.POINTER(C.c_int64), C.POINTER(C.c_double)]
    lib.lagkv_keep_for_compression.restype = C.c_int
    lib.lagkv_workspace_bytes.argtypes = [C.POINTER(Params), i64]
    lib.lagkv_workspace_bytes.restype = sz
    lib.lagkv_score.argtypes = [C.POINTER(Params), vp, vp, i64, vp, vp, sz, vp]
    lib.lagkv_score.restype = C.c_int
    lib.lagkv_select.argtypes = [C.POINTER(Params), vp, i64, vp, vp]
    lib.lagkv_select.restype = C.c_int
    lib.lagkv_compress.argtypes = [C.POINTER(Params), vp, vp, i64, vp, vp, vp, vp, vp, sz, vp]
    lib.lagkv_compress.restype = C.c_int
    lib.lagkv_append_and_compress.argtypes = [C.POINTER(Params), C.POINTER(CacheT), vp, vp, i64, vp,
                                              sz, vp]
    lib.lagkv_append_and_compress.restype = C.c_int
    lib.lagkv_compress_static.argtypes = [C.POINTER(Params), vp, vp, i64, vp, vp, vp, vp, vp]
    lib.lagkv_compress_static.restype = C.c_int
    lib.lagkv_cache_after_compress.argtypes = [C.POINTER(Params), i64, C.POINTER(CacheT)]
    lib.lagkv_cache_after_compress.restype = C.c_int
    lib.lagkv_prefill_rows.argtypes = [C.POINTER(Params), C.POINTER(CacheT), i64]
    lib.lagkv_prefill_rows.restype = C.c_int64
    lib.lagkv_prefill.argtypes = [C.POINTER(Params), C.POINTER(CacheT), vp, vp, i64, vp, sz, vp, C.POINTER(i64)]
    lib.lagkv_prefill.restype = C.c_int
    lib.lagkv_launch_hint.argtypes = [C.c_int, C.c_int, C.c_int]
    lib.lagkv_launch_hint.restype = C.c_int32
    lib.lagkv_launch_hint_ex.argtypes = [C.c_int] * 5
    lib.lagkv_launch_hint_ex.restype = C.c_int32
    lib.lagkv_path_for.argtypes = [C.POINTER(Params), C.c_int64]
    lib.lagkv_path_for.restype = C.c_int
    lib.lagkv_kernel_for.argtypes = [C.POINTER(Params), C.c_int64]
    lib.lagkv_kernel_for.restype = C.c_char_p
    lib.lagkv_strerror.argtypes = [C.c_int]
    lib.lagkv_strerror.restype = C.c_char_p
    lib.lagkv_version.argtypes = []
    lib.lagkv_version.restype = C.c_int
    _lib = lib
    _native = _load_native(lib)
    return lib


def _load_native(lib):
    """csrc/binding.cpp's module, set up; None where it is not built, or with a torch that has no devices to call it on."""
    raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    if raw_stream is None:
        return None
    try:
        native = importlib.import_module("._lagkv_native", __package__)
    except ModuleNotFoundError:
        return None
    except ImportError as e:  # built for another torch or Python
        warnings.warn(f"_lagkv_native.so does not load and calls go through ctypes, some microseconds more each: {e}", RuntimeWarning)
        return None
    native.init(*(C.cast(f, C.c_void_p).value for f in (lib.lagkv_plan, lib.lagkv_workspace_bytes, lib.lagkv_compress,
                                                        lib.lagkv_append_and_compress)), raw_stream)
    return native


def strerror(status: int) -> str:
    return load().lagkv_strerror(int(status)).decode()


def version() -> int:
    return load().lagkv_version()


def _check(status: int, where: str):
    if status != OK:
        raise LagKVError(status, where)


_DTYPES = {torch.float32: F32, torch.bfloat16: BF16, torch.float16: F16}


def path_for(p: "Params", T: int) -> int:
    """lagkv_path_for: the PATH_* lagkv_compress takes for these parameters."""
    v = load().lagkv_path_for(C.byref(p), T)
    if v < 0:
        raise LagKVError(-v, "lagkv_path_for")
    return v


def kernel_for(p: "Params", T: int) -> str:
    """lagkv_kernel_for: name of the kernel that scores in a lagkv_compress call with these parameters."""
    name = load().lagkv_kernel_for(C.byref(p), T)
    if name is None:
        path_for(p, T)  # (raises with the status)
        raise LagKVError(EINVAL, "lagkv_kernel_for")
    return name.decode()


def launch_hint(path: int = PATH_AUTO, waves: int = 0, segments: int = 0, order: int = 0,
                select: int = 0) -> int:
    """lagkv_launch_hint(_ex): the value of Params.launch that overrides the launch choice of one call."""
    v = load().lagkv_launch_hint_ex(path, waves, segments, order, select) if (order or select) \
        else load().lagkv_launch_hint(path, waves, segments)
    if v < 0:
        raise LagKVError(EINVAL, "lagkv_launch_hint")
    return v


def make_params(B: int, H: int, D: int, S: int, L: int, r: float, dtype=BF16, variant=SCORE_LAG,
                std_ddof: int = 1, strides: Tuple[int, int, int] = (0, 0, 0), launch: int = 0) -> Params:
    if isinstance(dtype, torch.dtype):
        dtype = _DTYPES[dtype]
    return Params(B, H, D, S, L, float(r), dtype, variant, std_ddof, launch, *strides)


def params_for(K: torch.Tensor, S: int, L: int, r: float, variant=SCORE_LAG, std_ddof: int = 1,
               launch: int = 0) -> Params:
    """Parameters for a [B,H,T,D] tensor (any strides with a contiguous channel axis)."""
    if K.dim() != 4 or K.stride(3) != 1:
        raise ValueError("expected a [B,H,T,D] tensor with contiguous channels")
    if K.dtype not in _DTYPES:
        raise TypeError(f"unsupported dtype {K.dtype}")
    B, H, _, D = K.shape
    return make_params(B, H, D, S, L, r, _DTYPES[K.dtype], variant, std_ddof,
                       (K.stride(0), K.stride(1), K.stride(2)), launch)


def plan(p: Params, T: int, n_static: int = -1) -> PlanT:
    out = PlanT()
    _check(load().lagkv_plan(C.byref(p), T, n_static, C.byref(out)), "lagkv_plan")
    return out


def keep_for_compression(T: int, S: int, L: int, ratio: float) -> Tuple[int, float]:
    """lagkv_keep_for_compression: (k, r) reaching compression ratio >= `ratio` at fixed S, L."""
    k, r = C.c_int64(), C.c_double()
    _check(load().lagkv_keep_for_compression(T, S, L, ratio, C.byref(k), C.byref(r)),
           "lagkv_keep_for_compression")
    return int(k.value), float(r.value)


def workspace_bytes(p: Params, T: int) -> int:
    return int(load().lagkv_workspace_bytes(C.byref(p), T))


def _stream_ptr(device) -> int:
    if device.type != "cuda" or device.index is None:
        return torch.cuda.current_stream(device).cuda_stream  # (which refuses other devices)
    return torch._C._cuda_getCurrentRawStream(device.index)  # (the raw handle: no Stream object built for it)


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _same_layout(K: torch.Tensor, V: torch.Tensor):
    if V.shape != K.shape or V.stride() != K.stride() or V.dtype != K.dtype or V.device != K.device:
        raise ValueError("K and V must share shape, strides, dtype and device")


@functools.lru_cache(maxsize=512)
def _prepared(shape, strides, dtype, S: int, L: int, r: float, variant: int, std_ddof: int, launch: int):
    """What a one-shot call works out from values alone (never from a tensor's address): parameters, a
    reference to them, the plan and the workspace size.  A serving loop repeats the same few shapes, and
    building the structures and asking the library twice is a third of the time of a short call.  The
    entries are only read; callers get copies of the plan."""
    p = make_params(shape[0], shape[1], shape[3], S, L, r, _DTYPES[dtype], variant, std_ddof, strides[:3], launch)
    T = shape[2]
    pl = plan(p, T)
    return p, C.byref(p), pl, _compress_bytes(p, T, pl)


def _compress_bytes(p: Params, T: int, pl: PlanT) -> int:
    """Workspace of one lagkv_compress call (see lagkv_workspace_bytes in include/lagkv.h): its scores and kept
    positions, without the two staged copies of a whole cache that an append may need."""
    if workspace_bytes(p, T) == 0:
        return 0
    return sum((4 * p.B * p.H * pl.n_scored * n + 255) // 256 * 256 for n in (p.L, pl.k))


def _prepare(K: torch.Tensor, S, L, r, variant, std_ddof, launch):
    strides = K.stride()
    if K.dim() != 4 or strides[3] != 1:
        raise ValueError("expected a [B,H,T,D] tensor with contiguous channels")
    if K.dtype not in _DTYPES:
        raise TypeError(f"unsupported dtype {K.dtype}")
    return _prepared(K.shape, strides, K.dtype, index(S), index(L), float(r), index(variant), index(std_ddof),
                     index(launch))


def score(K: torch.Tensor, V: Optional[torch.Tensor], S: int, L: int, r: float, variant=SCORE_LAG,
          std_ddof: int = 1, ws: Optional[torch.Tensor] = None, launch: int = 0) -> torch.Tensor:
    """lagkv_score: fp32 scores [B,H,n_scored*L] of every scored chunk."""
    if not K.is_cuda:
        raise RuntimeError("lagkv.score needs device tensors; there is no CPU path")
    if V is not None:
        _same_layout(K, V)
    p, ref, pl, _ = _prepare(K, S, L, r, variant, std_ddof, launch)
    T = K.shape[2]
    out = torch.empty((p.B, p.H, pl.n_scored * L), dtype=torch.float32, device=K.device)
    _check(load().lagkv_score(ref, K.data_ptr(), _ptr(V), T, out.data_ptr(), _ptr(ws),
                              0 if ws is None else ws.numel(), _stream_ptr(K.device)), "lagkv_score")
    return out


def select(scores: torch.Tensor, T: int, S: int, L: int, r: float) -> torch.Tensor:
    """lagkv_select: int32 kept positions [B,H,n_scored,k], ascending per chunk."""
    if not scores.is_cuda:
        raise RuntimeError("lagkv.select needs device tensors; there is no CPU path")
    if scores.dim() != 3 or not scores.is_contiguous() or scores.dtype != torch.float32:
        raise ValueError("scores must be a dense fp32 [B,H,n_scored*L] tensor")
    B, H, _ = scores.shape
    _, ref, pl, _ = _prepared((B, H, index(T), 2), (0, 0, 0), torch.float32, index(S), index(L), float(r), SCORE_LAG, 1, 0)
    if scores.shape[2] != pl.n_scored * L:
        raise ValueError("scores do not match the partition of T")
    kept = torch.empty((B, H, pl.n_scored, pl.k), dtype=torch.int32, device=scores.device)
    _check(load().lagkv_select(ref, scores.data_ptr(), T, kept.data_ptr(),
                               _stream_ptr(scores.device)), "lagkv_select")
    return kept


@dataclass
class Compressed:
    K: torch.Tensor                 # [B,H,T_out,D]
    V: torch.Tensor
    idx: Optional[torch.Tensor]     # [B,H,T_out] int32 source rows
    scores: Optional[torch.Tensor]  # [B,H,n_scored*L] fp32
    plan: PlanT


def compress(K: torch.Tensor, V: torch.Tensor, S: int, L: int, r: float, variant=SCORE_LAG,
             std_ddof: int = 1, want_idx: bool = True, want_scores: bool = False,
             out: Optional[Tuple[torch.Tensor, torch.Tensor]] = None,
             idx_out: Optional[torch.Tensor] = None, scores_out: Optional[torch.Tensor] = None,
             ws: Optional[torch.Tensor] = None, launch: int = 0) -> Compressed:
    """lagkv_compress: one whole pass.  Output buffers may be passed in (benchmarks)."""
    if _native is not None and out is None and idx_out is None and scores_out is None and ws is None:
        got = _native.compress(K, V, S, L, r, variant, std_ddof, launch, want_idx, want_scores)
        if isinstance(got, int):
            raise LagKVError(got, "lagkv_compress")
        if got is not None:
            return Compressed(got[0], got[1], got[2], got[3], PlanT.from_buffer_copy(got[4]))
    if not K.is_cuda:
        raise RuntimeError("lagkv.compress needs device tensors; there is no CPU path")
    _same_layout(K, V)
    p, ref, pl, need = _prepare(K, S, L, r, variant, std_ddof, launch)
    B, H, T, D = K.shape
    device = K.device
    if out is None:
        Ko = torch.empty((B, H, pl.T_out, D), dtype=K.dtype, device=device)
        Vo = torch.empty((B, H, pl.T_out, D), dtype=K.dtype, device=device)
    else:
        Ko, Vo = out
        if tuple(Ko.shape) != (B, H, pl.T_out, D) or not Ko.is_contiguous() or not Vo.is_contiguous() \
                or Vo.shape != Ko.shape or Ko.dtype != K.dtype or Vo.dtype != K.dtype:
            raise ValueError("output buffers must be dense [B,H,T_out,D] of the input dtype")
    if idx_out is None and want_idx:
        idx_out = torch.empty((B, H, pl.T_out), dtype=torch.int32, device=device)
    if scores_out is None and want_scores:
        scores_out = torch.empty((B, H, pl.n_scored * L), dtype=torch.float32, device=device)
    if ws is None and need:
        ws = torch.empty(need, dtype=torch.uint8, device=device)
    _check(load().lagkv_compress(ref, K.data_ptr(), V.data_ptr(), T, Ko.data_ptr(),
                                 Vo.data_ptr(), _ptr(idx_out), _ptr(scores_out), _ptr(ws),
                                 0 if ws is None else ws.numel(), _stream_ptr(device)),
           "lagkv_compress")
    return Compressed(Ko, Vo, idx_out, scores_out, PlanT.from_buffer_copy(pl))


STATIC_SCRATCH_BYTES = 16 << 20


def compress_static(K: torch.Tensor, V: torch.Tensor, S: int, L: int, r: float, out: Tuple[torch.Tensor, torch.Tensor],
                    idx_out: Optional[torch.Tensor] = None, scores_out: Optional[torch.Tensor] = None,
                    variant=SCORE_LAG, std_ddof: int = 1, launch: int = 0) -> PlanT:
    """lagkv_compress_static: the whole pass into caller-provided buffers with no workspace and no
    allocation anywhere (the three-kernel path stages in the library's static device array)."""
    if not K.is_cuda:
        raise RuntimeError("lagkv.compress_static needs device tensors; there is no CPU path")
    _same_layout(K, V)
    p = params_for(K, S, L, r, variant, std_ddof, launch)
    B, H, T, D = K.shape
    pl = plan(p, T)
    Ko, Vo = out
    if tuple(Ko.shape) != (B, H, pl.T_out, D) or not Ko.is_contiguous() or not Vo.is_contiguous() \
            or Vo.shape != Ko.shape or Ko.dtype != K.dtype or Vo.dtype != K.dtype:
        raise ValueError("output buffers must be dense [B,H,T_out,D] of the input dtype")
    _check(load().lagkv_compress_static(C.byref(p), K.data_ptr(), V.data_ptr(), T, Ko.data_ptr(),
                                        Vo.data_ptr(), _ptr(idx_out), _ptr(scores_out),
                                        _stream_ptr(K.device)), "lagkv_compress_static")
    return pl


class Cache:
    """Caller-owned decode-time cache: dense [B,H,capacity,D] buffers + the host
    counters of lagkv_cache.  `append_and_compress` forwards to the C call."""

    def __init__(self, B: int, H: int, D: int, capacity: int, S: int, L: int, r: float,
                 dtype=torch.bfloat16, device="cuda", variant=SCORE_LAG, std_ddof: int = 1,
                 track_positions: bool = True, launch: int = 0):
        self.S, self.L, self.r, self.variant, self.std_ddof = S, L, r, variant, std_ddof
        self.launch = launch
        self.K = torch.empty((B, H, capacity, D), dtype=dtype, device=device)
        self.V = torch.empty_like(self.K)
        self.pos = torch.empty((B, H, capacity), dtype=torch.int32, device=device) \
            if track_positions else None
        self.c = CacheT(self.K.data_ptr(), self.V.data_ptr(), _ptr(self.pos), capacity, 0, 0, 0)
        self._ws = None
        self._prepared = {}

    @classmethod
    def from_compressed(cls, comp: Compressed, T: int, capacity: int, S: int, L: int, r: float,
                        variant=SCORE_LAG, std_ddof: int = 1, launch: int = 0) -> "Cache":
        """Cache holding the output of compress() on T rows, with room to grow."""
        B, H, T_out, D = comp.K.shape
        c = cls(B, H, D, capacity, S, L, r, comp.K.dtype, comp.K.device, variant, std_ddof,
                comp.idx is not None, launch)
        c.K[:, :, :T_out].copy_(comp.K)
        c.V[:, :, :T_out].copy_(comp.V)
        if comp.idx is not None:
            c.pos[:, :, :T_out].copy_(comp.idx)
        c.mark_compressed(T)
        return c

    def _params(self, strides=(0, 0, 0)) -> Params:
        B, H, _, D = self.K.shape
        return make_params(B, H, D, self.S, self.L, self.r, _DTYPES[self.K.dtype], self.variant,
                           self.std_ddof, strides, self.launch)

    def mark_compressed(self, T: int) -> None:
        """lagkv_cache_after_compress: the buffers now hold the output of compress() on T rows."""
        _check(load().lagkv_cache_after_compress(C.byref(self._params()), T, C.byref(self.c)),
               "lagkv_cache_after_compress")

    @property
    def n_static(self) -> int:
        return self.c.n_static

    @property
    def n_tail(self) -> int:
        return self.c.n_tail

    @property
    def n_seen(self) -> int:
        return self.c.n_seen

    @property
    def length(self) -> int:
        return self.c.n_static + self.c.n_tail

    def _prepare(self, strides):
        """Parameters and workspace size of a call whose new rows have these strides (0: dense).  They depend on
        values only - the cache's own, which are part of the key, and the strides; the last few are kept."""
        key = (strides, self.K.shape, self.K.dtype, self.S, self.L, self.r, self.variant, self.std_ddof, self.launch)
        got = self._prepared.get(key)
        if got is None:
            if len(self._prepared) >= 64:
                self._prepared = {}
            p = self._params(strides)
            got = self._prepared[key] = (p, C.byref(p), workspace_bytes(p, self.K.shape[2]))
        return got

    def _workspace(self, need: int) -> Optional[torch.Tensor]:
        if need > 0 and (self._ws is None or self._ws.numel() < need):
            self._ws = torch.empty(need, dtype=torch.uint8, device=self.K.device)
        return self._ws

    def append_and_compress(self, K_new: Optional[torch.Tensor], V_new: Optional[torch.Tensor]) -> None:
        K = self.K
        if _native is not None:
            rc = _native.append(self.c, K, self.S, self.L, self.r, self.variant, self.std_ddof, self.launch, self._ws, K_new, V_new)
            if rc == OK:
                return
            if rc > 0:
                raise LagKVError(rc, "lagkv_append_and_compress")
        if K_new is None:
            n_new, strides = 0, (0, 0, 0)
        else:
            _same_layout(K_new, V_new)
            shape, have, strides = K_new.shape, K.shape, K_new.stride()
            if len(shape) != 4 or strides[3] != 1 or shape[0] != have[0] or shape[1] != have[1] \
                    or shape[3] != have[3] or K_new.dtype != K.dtype:
                raise ValueError("K_new must be [B,H,n_new,D] of the cache dtype")
            n_new, strides = shape[2], strides[:3]
        p, ref, need = self._prepare(strides)
        ws = self._workspace(need) if need else self._ws
        _check(load().lagkv_append_and_compress(
            ref, C.byref(self.c), _ptr(K_new), _ptr(V_new), n_new, _ptr(ws),
            0 if ws is None else ws.numel(), _stream_ptr(K.device)),
            "lagkv_append_and_compress")

    def prefill_chunked(self, K: torch.Tensor, V: torch.Tensor) -> int:
        """Chunk-by-chunk compression during prefill (Ablation, subsection on the prefill
        stage): the first S + 2L rows in one call, then L rows per call until all rows
        are in; every call is lagkv_append_and_compress.  The model forward that would produce
        each slice between the calls is the caller's; here the rows are given, and
        lagkv_prefill makes the calls, or on an empty cache one pass in their place.  Returns the
        number of calls."""
        T, have = K.shape[2], self.K.shape
        strides = K.stride()
        if T and isinstance(V, torch.Tensor) and K.shape == (have[0], have[1], T, have[3]) and strides[3] == 1 \
                and 0 not in strides and (V.shape, V.stride(), V.dtype, V.device) == (K.shape, strides, K.dtype, K.device) \
                and (K.dtype, K.device) == (self.K.dtype, self.K.device):
            _, ref, need = self._prepare(strides[:3])
            calls = C.c_int64()
            _check(load().lagkv_prefill(ref, C.byref(self.c), K.data_ptr(), V.data_ptr(), T, _ptr(self._workspace(need)), need,
                                        _stream_ptr(self.K.device), C.byref(calls)), "lagkv_append_and_compress")
            return calls.value
        # (what is wrong with the rows is said by the call that meets it, as the calls before it have been made)
        p = self._params()
        calls, t = 0, 0
        while t < T:
            n = load().lagkv_prefill_rows(C.byref(p), C.byref(self.c), T - t)
            if n <= 0:
                raise LagKVError(EINVAL, "lagkv_prefill_rows")
            self.append_and_compress(K[:, :, t:t + n], V[:, :, t:t + n])
            t += n
            calls += 1
        return calls

    def view(self) -> Tuple[torch.Tensor, torch.Tensor, Optional[torch.Tensor]]:
        n = self.length
        return self.K[:, :, :n], self.V[:, :, :n], None if self.pos is None else self.pos[:, :, :n]
