"""Thin binding of ``libngc.so`` (see ``include/ngc.h``).

Argument marshalling only: every step of the path runs in the HIP kernels.  The
calls that enqueue work go through ``_ngc_host.so`` (``csrc/ngc_host.cpp``),
which reads the tensors' pointers and calls the C ABI; ``load_library`` also
gives the library as a ctypes object for callers that prepare the C arguments
themselves.
PyTorch tensors are used as device memory and for the current HIP stream; no
torch operator takes part in the computation.  There is no CPU fallback: a
missing library raises.
"""
from __future__ import annotations

import ctypes as C
import os
import sys
from dataclasses import dataclass
from typing import Optional

from ._build import HOST_LIB_PATH, LIB_PATH, TORCH_LIB_PATH, torch_identity

NGC_OK = 0
NGC_EINVAL = -1
NGC_ENOSPC = -2
NGC_EHIP = -3
NGC_EUNSUPPORTED = -4

STATUS_WORDS = 64
STATUS_KEEP_CLAMPED = 0
STATUS_LEN_CLAMPED = 1
STATUS_EMPTY_ATTN = 2
STATUS_APPEND_FULL = 3
STATUS_BAD_SIGMA = 4
STATUS_POOL_BOUNDS = 5

EVICT_SELECT_ONLY = 1
EVICT_UNORDERED = 2
EVICT_POOL_HEADS = 4
SCORE_NO_CAUSAL = 1
SCORE_POOL_HEADS = 2

EXPORTS = ("ngc_version", "ngc_strerror", "ngc_workspace_bytes", "ngc_perturbed_keys", "ngc_evict",
           "ngc_subset_logprob", "ngc_cache_append", "ngc_decode_attn", "ngc_score_keys",
           "ngc_subset_logprob_backward", "ngc_replay_attn", "ngc_replay_workspace_bytes",
           "ngc_paged_workspace_bytes", "ngc_paged_evict", "ngc_paged_append", "ngc_paged_decode_attn",
           "ngc_paged_score_keys", "ngc_lmem", "ngc_keep_counts", "ngc_decode_attn_static", "ngc_decode_step")
STATIC_SCRATCH_BYTES = 2 << 20


class NgcError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {strerror(code)} ({code})")


class ArgumentError(C.ArgumentError, TypeError):
    """An argument of the wrong type."""


class ngc_cache(C.Structure):
    _fields_ = [("k", C.c_void_p), ("v", C.c_void_p), ("len", C.c_void_p), ("pos", C.c_void_p),
                ("L", C.c_int32), ("B", C.c_int32), ("Hkv", C.c_int32), ("Hq", C.c_int32),
                ("D", C.c_int32), ("cap", C.c_int32)]


class ngc_paged_cache(C.Structure):
    _fields_ = [("k_pool", C.c_void_p), ("v_pool", C.c_void_p), ("pos_pool", C.c_void_p),
                ("table", C.c_void_p), ("len", C.c_void_p), ("free_stack", C.c_void_p),
                ("free_count", C.c_void_p),
                ("L", C.c_int32), ("B", C.c_int32), ("Hkv", C.c_int32), ("Hq", C.c_int32), ("D", C.c_int32),
                ("page_rows", C.c_int32), ("max_pages", C.c_int32), ("num_pages", C.c_int32)]


class ngc_evict_params(C.Structure):
    _fields_ = [("block", C.c_int32), ("share_heads", C.c_int32), ("noise_scale", C.c_float),
                ("round", C.c_uint32), ("seed", C.c_uint64), ("flags", C.c_uint32),
                ("layer_base", C.c_int32), ("seq_base", C.c_int32), ("reserved", C.c_int32)]


_lib = None
_host = None      # the CPython front, opened on the same library


def load_library(path: Optional[str] = None) -> C.CDLL:
    """Load the built library.  Raises if it has not been built."""
    global _lib, _host
    if _lib is not None and path is None:
        return _lib
    path = path or LIB_PATH
    # PyTorch ships its own copy of the HIP runtime.  It has to be in the process before this library
    # pulls in the system's, or the two runtimes would not share streams and launches on torch's streams fail.
    try:
        import torch  # noqa: F401
    except ImportError:
        pass
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is missing: build it first (python -m paper_2604_18002_amd._build); "
                           "there is no fallback path")
    lib = C.CDLL(path)
    vp, i32, i64, f32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_float, C.c_size_t
    cp, pp = C.POINTER(ngc_cache), C.POINTER(ngc_evict_params)
    lib.ngc_version.argtypes = []
    lib.ngc_version.restype = C.c_int
    lib.ngc_strerror.argtypes = [C.c_int]
    lib.ngc_strerror.restype = C.c_char_p
    lib.ngc_workspace_bytes.argtypes = [cp, i32]
    lib.ngc_workspace_bytes.restype = sz
    lib.ngc_perturbed_keys.argtypes = [cp, i32, vp, pp, vp, vp, sz, vp]
    lib.ngc_perturbed_keys.restype = C.c_int
    lib.ngc_evict.argtypes = [cp, i32, vp, vp, pp, i32, vp, vp, vp, vp, sz, vp]
    lib.ngc_evict.restype = C.c_int
    lib.ngc_subset_logprob.argtypes = [vp, vp, vp, vp, i32, i64, i32, vp, vp, sz, vp]
    lib.ngc_subset_logprob.restype = C.c_int
    lib.ngc_cache_append.argtypes = [cp, i32, vp, vp, vp, vp, sz, vp]
    lib.ngc_cache_append.restype = C.c_int
    lib.ngc_decode_attn.argtypes = [cp, i32, vp, f32, i32, vp, vp, vp, sz, vp]
    lib.ngc_decode_attn.restype = C.c_int
    lib.ngc_decode_step.argtypes = [cp, i32, vp, vp, vp, vp, f32, i32, vp, vp, vp, sz, vp]
    lib.ngc_decode_step.restype = C.c_int
    lib.ngc_decode_attn_static.argtypes = [cp, i32, vp, f32, i32, vp, vp, vp, vp]
    lib.ngc_decode_attn_static.restype = C.c_int
    lib.ngc_subset_logprob_backward.argtypes = [vp, vp, vp, vp, i32, i64, i32, i32, vp, vp, vp, sz, vp]
    lib.ngc_subset_logprob_backward.restype = C.c_int
    lib.ngc_replay_workspace_bytes.argtypes = [i32, i32, i32]
    lib.ngc_replay_workspace_bytes.restype = sz
    lib.ngc_replay_attn.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, f32, vp, vp, sz, vp]
    lib.ngc_replay_attn.restype = C.c_int
    lib.ngc_score_keys.argtypes = [cp, i32, vp, vp, i32, f32, C.c_uint32, i32, vp, vp, sz, vp]
    lib.ngc_score_keys.restype = C.c_int
    gp = C.POINTER(ngc_paged_cache)
    lib.ngc_paged_workspace_bytes.argtypes = [gp]
    lib.ngc_paged_workspace_bytes.restype = sz
    lib.ngc_paged_evict.argtypes = [gp, i32, vp, i64, vp, pp, i32, vp, vp, vp, vp, sz, vp]
    lib.ngc_paged_evict.restype = C.c_int
    lib.ngc_paged_append.argtypes = [gp, i32, vp, vp, vp, vp, sz, vp]
    lib.ngc_paged_append.restype = C.c_int
    lib.ngc_paged_decode_attn.argtypes = [gp, i32, vp, f32, i32, vp, vp, vp, sz, vp]
    lib.ngc_paged_decode_attn.restype = C.c_int
    lib.ngc_paged_score_keys.argtypes = [gp, i32, vp, vp, i32, f32, C.c_uint32, i32, vp, vp, sz, vp]
    lib.ngc_paged_score_keys.restype = C.c_int
    lib.ngc_lmem.argtypes = [vp, vp, vp, i32, i32, i32, i32, i32, vp, vp, vp, vp, vp]
    lib.ngc_lmem.restype = C.c_int
    lib.ngc_keep_counts.argtypes = [vp, i32, i32, i32, i32, i32, i32, i32, vp, vp]
    lib.ngc_keep_counts.restype = C.c_int
    if path == LIB_PATH:
        if not os.path.exists(HOST_LIB_PATH):
            raise RuntimeError(f"{HOST_LIB_PATH} is missing: build it first (python -m paper_2604_18002_amd._build); "
                               "there is no fallback path")
        from . import _ngc_host
        _ngc_host.open(path)
        _ngc_host.types(ArgumentError, Cache, PagedCache, ngc_cache, ngc_paged_cache, ngc_evict_params, C._SimpleCData)
        _read_tensors_directly(_ngc_host)
        _host = _ngc_host
        _lib = lib
    return lib


def _read_tensors_directly(host) -> bool:
    """From now on the front reads plain tensors itself, if torch has been imported and the reader was compiled against
    this very torch; otherwise it asks the tensors' methods, which takes longer and gives the same."""
    torch = sys.modules.get("torch")
    if getattr(torch, "_C", None) is None or not hasattr(torch, "version"):     # (absent, blocked, or still being imported)
        return False
    return host.torch_reader(TORCH_LIB_PATH, torch_identity(torch))


def _front():
    """The CPython front (loads the library on first use)."""
    if _host is None:
        load_library()
    return _host


def strerror(code: int) -> str:
    return load_library().ngc_strerror(code).decode()


def version() -> int:
    return load_library().ngc_version()


def _ptr(t) -> Optional[int]:
    return None if t is None else t.data_ptr()


_current_raw_stream = None


def _forget_stream_reader() -> None:
    """A forked child asks torch again, which refuses there if the parent had initialised the GPU."""
    global _current_raw_stream
    _current_raw_stream = None


os.register_at_fork(after_in_child=_forget_stream_reader)


def _stream(stream) -> Optional[int]:
    if stream is not None:
        return stream if isinstance(stream, int) else stream.cuda_stream
    global _current_raw_stream
    if _current_raw_stream is None:
        import torch
        torch.cuda.current_stream()     # initialises the runtime (or says why it cannot)
        # the current stream of the current device, without the Stream object where torch has its own way to that
        get, device = (getattr(torch._C, name, None) for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"))
        if get and device:
            host = _front()
            _read_tensors_directly(host)        # (torch may have been imported after the library)
            host.stream_readers(device, get)
            _current_raw_stream = host.current_stream
        else:
            _current_raw_stream = lambda: torch.cuda.current_stream().cuda_stream     # noqa: E731
    return _current_raw_stream()


def _check(rc: int, where: str) -> None:
    if rc != NGC_OK:
        raise NgcError(rc, where)


@dataclass
class Cache:
    """Device buffers of a KV cache (torch tensors as plain memory).

    k, v: bf16 [L, B, Hkv, cap, D]; len: int32 [L, B, Hkv]; pos: int32 [L, B, Hkv, cap] or None."""
    k: object
    v: object
    len: object
    pos: object
    Hq: int

    @property
    def shape(self):
        L, B, Hkv, cap, D = self.k.shape
        return L, B, Hkv, cap, D

    def view(self) -> ngc_cache:
        L, B, Hkv, cap, D = self.k.shape
        assert self.k.is_contiguous() and self.v.is_contiguous() and self.len.is_contiguous()
        return ngc_cache(_ptr(self.k), _ptr(self.v), _ptr(self.len), _ptr(self.pos), L, B, Hkv, self.Hq, D, cap)

    @staticmethod
    def allocate(L, B, Hkv, Hq, D, cap, device="cuda", with_pos=False) -> "Cache":
        import torch
        k = torch.zeros(L, B, Hkv, cap, D, dtype=torch.bfloat16, device=device)
        v = torch.zeros_like(k)
        ln = torch.zeros(L, B, Hkv, dtype=torch.int32, device=device)
        pos = torch.zeros(L, B, Hkv, cap, dtype=torch.int32, device=device) if with_pos else None
        return Cache(k, v, ln, pos, Hq)


def make_params(block=1, share_heads=0, noise_scale=1.0, round=0, seed=0, flags=0, layer_base=0,
                seq_base=0) -> ngc_evict_params:
    return ngc_evict_params(block, share_heads, noise_scale, round, seed, flags, layer_base, seq_base, 0)


def ngc_workspace_bytes(cache: Cache, max_keep: int) -> int:
    v = cache.view()
    return int(load_library().ngc_workspace_bytes(C.byref(v), max_keep))


def allocate_workspace(cache: Cache, max_keep: int):
    """A zeroed workspace tensor (uint8) of the size the library asks for."""
    import torch
    return torch.zeros(ngc_workspace_bytes(cache, max_keep), dtype=torch.uint8, device=cache.k.device)


def read_status(ws):
    """Status counters at the start of a workspace (copies to host, synchronises)."""
    return ws[:STATUS_WORDS * 4].view(dtype=_i32()).cpu().tolist()


def _i32():
    import torch
    return torch.int32


def ngc_perturbed_keys(cache: Cache, layer: int, logits, params: ngc_evict_params, keys_out, ws, stream=None):
    _check(_front().perturbed_keys(cache, layer, logits, params, keys_out, ws, _stream(stream)),
           "ngc_perturbed_keys")


def ngc_evict(cache: Cache, layer: int, logits, keep, params: ngc_evict_params, max_keep: int,
              kept_out, sigma_out, logp_out, ws, stream=None):
    _check(_front().evict(cache, layer, logits, keep, params, max_keep, kept_out, sigma_out, logp_out, ws,
                          _stream(stream)),
           "ngc_evict")


def ngc_subset_logprob(logits, n_items, sigma, keep, nseg: int, logit_stride: int, sigma_stride: int,
                       logp_out, ws, stream=None):
    _check(_front().subset_logprob(logits, n_items, sigma, keep, nseg, logit_stride, sigma_stride, logp_out, ws,
                                   _stream(stream)),
           "ngc_subset_logprob")


def ngc_cache_append(cache: Cache, layer: int, k_new, v_new, new_pos, ws, stream=None):
    _check(_front().cache_append(cache, layer, k_new, v_new, new_pos, ws, _stream(stream)),
           "ngc_cache_append")


def ngc_decode_attn(cache: Cache, layer: int, q, scale: float, max_len_hint: int, out, ws, stream=None,
                    lse_out=None):
    _check(_front().decode_attn(cache, layer, q, scale, max_len_hint, out, lse_out, ws, _stream(stream)),
           "ngc_decode_attn")


def ngc_decode_step(cache: Cache, layer: int, k_new, v_new, new_pos, q, scale: float, max_len_hint: int, out, ws,
                    stream=None, lse_out=None):
    _check(_front().decode_step(cache, layer, k_new, v_new, new_pos, q, scale, max_len_hint, out, lse_out, ws,
                                _stream(stream)),
           "ngc_decode_step")


def ngc_decode_attn_static(cache: Cache, layer: int, q, scale: float, max_len_hint: int, out, stream=None,
                           lse_out=None, status=None):
    _check(_front().decode_attn_static(cache, layer, q, scale, max_len_hint, out, lse_out, status,
                                       _stream(stream)),
           "ngc_decode_attn_static")


def ngc_score_keys(cache: Cache, layer: int, q_recent, w: int, scale: float, flags: int, block: int,
                   scores_out, ws, stream=None, lse_recent=None):
    _check(_front().score_keys(cache, layer, q_recent, lse_recent, w, scale, flags, block, scores_out, ws,
                               _stream(stream)),
           "ngc_score_keys")


def ngc_subset_logprob_backward(logits, n_items, sigma, keep, nseg: int, logit_stride: int, sigma_stride: int,
                                max_keep: int, gout, grad_out, ws, stream=None):
    _check(_front().subset_logprob_backward(logits, n_items, sigma, keep, nseg, logit_stride, sigma_stride,
                                            max_keep, gout, grad_out, ws, _stream(stream)),
           "ngc_subset_logprob_backward")


def ngc_replay_workspace_bytes(B: int, T: int, Hkv: int) -> int:
    return int(load_library().ngc_replay_workspace_bytes(B, T, Hkv))


def ngc_replay_attn(q, k, v, death, B: int, T: int, Hq: int, Hkv: int, D: int, death_per_head: bool,
                    scale: float, out, ws, stream=None):
    _check(_front().replay_attn(q, k, v, death, B, T, Hq, Hkv, D, 1 if death_per_head else 0, scale, out, ws,
                                _stream(stream)),
           "ngc_replay_attn")


# ------------------------------------------------------------- paged layout ---

@dataclass
class PagedCache:
    """Device buffers of a paged KV cache (torch tensors as plain memory).

    k_pool, v_pool: bf16 [num_pages, page_rows, D]; pos_pool: int32 [num_pages, page_rows] or None;
    table: int32 [L, B, Hkv, max_pages]; len: int32 [L, B, Hkv]; free_stack: int32 [num_pages];
    free_count: int32 [1]."""
    k_pool: object
    v_pool: object
    pos_pool: object
    table: object
    len: object
    free_stack: object
    free_count: object
    Hq: int

    @property
    def page_rows(self) -> int:
        return self.k_pool.shape[1]

    @property
    def cap(self) -> int:
        return self.table.shape[3] * self.k_pool.shape[1]

    def view(self) -> ngc_paged_cache:
        num_pages, P, D = self.k_pool.shape
        L, B, Hkv, max_pages = self.table.shape
        for t in (self.k_pool, self.v_pool, self.table, self.len, self.free_stack, self.free_count):
            assert t.is_contiguous()
        return ngc_paged_cache(_ptr(self.k_pool), _ptr(self.v_pool), _ptr(self.pos_pool), _ptr(self.table),
                               _ptr(self.len), _ptr(self.free_stack), _ptr(self.free_count),
                               L, B, Hkv, self.Hq, D, P, max_pages, num_pages)

    @staticmethod
    def allocate(L, B, Hkv, Hq, D, page_rows, max_pages, num_pages, device="cuda", with_pos=False) -> "PagedCache":
        """An empty cache: every page on the free stack (page 0 on top)."""
        import torch
        k = torch.zeros(num_pages, page_rows, D, dtype=torch.bfloat16, device=device)
        v = torch.zeros_like(k)
        pos = torch.zeros(num_pages, page_rows, dtype=torch.int32, device=device) if with_pos else None
        table = torch.full((L, B, Hkv, max_pages), -1, dtype=torch.int32, device=device)
        ln = torch.zeros(L, B, Hkv, dtype=torch.int32, device=device)
        stack = torch.arange(num_pages - 1, -1, -1, dtype=torch.int32, device=device)
        count = torch.full((1,), num_pages, dtype=torch.int32, device=device)
        return PagedCache(k, v, pos, table, ln, stack, count, Hq)


def ngc_paged_workspace_bytes(pc: PagedCache) -> int:
    v = pc.view()
    return int(load_library().ngc_paged_workspace_bytes(C.byref(v)))


def allocate_paged_workspace(pc: PagedCache):
    import torch
    return torch.zeros(ngc_paged_workspace_bytes(pc), dtype=torch.uint8, device=pc.k_pool.device)


def ngc_paged_evict(pc: PagedCache, layer: int, logits, logit_stride: int, keep, params: ngc_evict_params,
                    max_keep: int, kept_out, sigma_out, logp_out, ws, stream=None):
    _check(_front().paged_evict(pc, layer, logits, logit_stride, keep, params, max_keep, kept_out, sigma_out,
                                logp_out, ws, _stream(stream)),
           "ngc_paged_evict")


def ngc_paged_append(pc: PagedCache, layer: int, k_new, v_new, new_pos, ws, stream=None):
    _check(_front().paged_append(pc, layer, k_new, v_new, new_pos, ws, _stream(stream)),
           "ngc_paged_append")


def ngc_paged_decode_attn(pc: PagedCache, layer: int, q, scale: float, max_len_hint: int, out, ws, stream=None,
                          lse_out=None):
    _check(_front().paged_decode_attn(pc, layer, q, scale, max_len_hint, out, lse_out, ws, _stream(stream)),
           "ngc_paged_decode_attn")


def ngc_paged_score_keys(pc: PagedCache, layer: int, q_recent, w: int, scale: float, flags: int, block: int,
                         scores_out, ws, stream=None, lse_recent=None):
    _check(_front().paged_score_keys(pc, layer, q_recent, lse_recent, w, scale, flags, block, scores_out, ws,
                                     _stream(stream)),
           "ngc_paged_score_keys")


def ngc_lmem(logp, rounds, reward, R: int, L: int, B: int, Hkv: int, group: int, adv_out, loss_layer, loss,
             gout, stream=None):
    _check(_front().lmem(logp, rounds, reward, R, L, B, Hkv, group, adv_out, loss_layer, loss, gout,
                         _stream(stream)),
           "ngc_lmem")


def ngc_keep_counts(len_t, seg0: int, nseg: int, cap: int, block: int, num: int, den: int, min_keep: int, keep_out,
                    stream=None):
    _check(_front().keep_counts(len_t, seg0, nseg, cap, block, num, den, min_keep, keep_out, _stream(stream)),
           "ngc_keep_counts")
