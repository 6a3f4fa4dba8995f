"""The CPython front of the C ABI (no GPU): what it reads from tensors arrives at the library, errors come back as before,
and nothing is called when reading an argument fails."""
import ctypes as C

import pytest
import torch

from paper_2604_18002_amd import binding as ngc


def _cache(L=2, B=3, H=2, Hq=12, D=128, cap=64):
    return ngc.Cache.allocate(L, B, H, Hq, D, cap, device="cpu")


def _code(call, *args, **kw):
    with pytest.raises(ngc.NgcError) as e:
        call(*args, stream=0, **kw)
    return e.value.code


def test_geometry_and_pointers_reach_the_library():
    """Argument checks that depend on one field each, against the same call through ctypes with the cache's own view."""
    lib = ngc.load_library()
    q, out = torch.zeros(3, 12, 128, dtype=torch.bfloat16), torch.zeros(3, 12, 128)
    ws = torch.zeros(1 << 20, dtype=torch.uint8)
    for kw, want in ((dict(Hq=13), ngc.NGC_EINVAL), (dict(Hq=64), ngc.NGC_EINVAL), (dict(D=96), ngc.NGC_EINVAL),
                     (dict(), ngc.NGC_EINVAL)):
        c = _cache(**kw)
        v = c.view()
        layer = 2 if not kw else 0          # a layer beyond the cache when the geometry itself is fine
        assert lib.ngc_decode_attn(C.byref(v), layer, q.data_ptr(), 0.1, 0, out.data_ptr(), None, ws.data_ptr(), ws.numel(),
                                   None) == want
        assert _code(ngc.ngc_decode_attn, c, layer, q, 0.1, 0, out, ws) == want
        assert _code(ngc.ngc_decode_step, c, layer, q, q, None, q, 0.1, 0, out, ws) == want
    c = _cache()
    assert _code(ngc.ngc_decode_attn, c, 0, q, float("nan"), 0, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_decode_attn, c, 0, q, 0.1, -1, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_decode_attn, c, 0, None, 0.1, 0, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_decode_attn, c, 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_ENOSPC
    assert _code(ngc.ngc_decode_attn, c, 0, q.view(-1)[1:], 0.1, 0, out, ws) == ngc.NGC_EINVAL       # misaligned
    assert _code(ngc.ngc_score_keys, c, 0, q, 65, 0.1, 0, 1, out, ws) == ngc.NGC_EUNSUPPORTED
    assert _code(ngc.ngc_score_keys, c, 0, q, 1, 0.1, ngc.SCORE_NO_CAUSAL, 1, out, ws, lse_recent=out) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_cache_append, c, 5, q, q, None, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_replay_attn, q, q, q, q, 1, 70000, 12, 2, 128, False, 0.1, out, ws) == ngc.NGC_EUNSUPPORTED
    assert _code(ngc.ngc_lmem, out, q, out, 1, 1, 10, 1, 3, None, out, out, None) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_keep_counts, q, 0, 4, 10, 1, 3, 2, 0, q) == ngc.NGC_EINVAL                  # num > den
    assert _code(ngc.ngc_subset_logprob, out, q, q, q, -1, 8, 8, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_subset_logprob_backward, out, q, q, q, 4, 10, 10, 40000, None, out, ws) == ngc.NGC_EUNSUPPORTED


def test_eviction_parameters_are_read_from_the_structure():
    c = _cache()
    x, keep = torch.zeros(2, 3, 2, 64), torch.zeros(2, 3, 2, dtype=torch.int32)
    kept, ws = torch.zeros(2, 3, 2, 8, dtype=torch.int32), torch.zeros(1 << 20, dtype=torch.uint8)

    def code(**kw):
        return _code(ngc.ngc_evict, c, 0, x, keep, ngc.make_params(**kw), 8, kept, None, None, ws)
    assert code(block=0) == ngc.NGC_EINVAL
    assert code(layer_base=65534) == ngc.NGC_EINVAL
    assert code(seq_base=-1) == ngc.NGC_EINVAL
    assert code(block=2, flags=ngc.EVICT_UNORDERED) == ngc.NGC_EUNSUPPORTED
    assert _code(ngc.ngc_perturbed_keys, c, 0, x, ngc.make_params(block=0), x, ws) == ngc.NGC_EINVAL
    with pytest.raises((TypeError, BufferError)):
        ngc.ngc_evict(c, 0, x, keep, None, 8, kept, None, None, ws, stream=0)
    with pytest.raises(TypeError):
        ngc.ngc_evict(c, 0, x, keep, b"short", 8, kept, None, None, ws, stream=0)


def test_paged_geometry_reaches_the_library():
    pc = ngc.PagedCache.allocate(2, 3, 2, 12, 128, 32, 4, 40, device="cpu")
    q, ws = torch.zeros(3, 12, 128, dtype=torch.bfloat16), torch.zeros(1 << 20, dtype=torch.uint8)
    out = torch.zeros(3, 12, 128)
    assert _code(ngc.ngc_paged_decode_attn, pc, 2, q, 0.1, 0, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_paged_append, pc, 0, q, q, None, ws[:8]) == ngc.NGC_ENOSPC
    assert _code(ngc.ngc_paged_score_keys, pc, 0, q, 65, 0.1, 0, 32, out, ws) == ngc.NGC_EUNSUPPORTED
    x, keep = torch.zeros(2, 3, 2, 4), torch.zeros(2, 3, 2, dtype=torch.int32)
    kept = torch.zeros(2, 3, 2, 4, dtype=torch.int32)
    assert _code(ngc.ngc_paged_evict, pc, 0, x, 4, keep, ngc.make_params(block=16), 4, kept, None, None, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_paged_evict, pc, 0, x, 3, keep, ngc.make_params(block=32), 4, kept, None, None, ws) == ngc.NGC_EINVAL
    odd = ngc.PagedCache.allocate(1, 1, 1, 1, 128, 48, 4, 8, device="cpu")      # page_rows not a power of two
    assert _code(ngc.ngc_paged_append, odd, 0, q, q, None, ws) == ngc.NGC_EINVAL


def test_unreadable_arguments_raise_and_call_nothing():
    c = _cache()
    q, out, ws = torch.zeros(3, 12, 128, dtype=torch.bfloat16), torch.zeros(3, 12, 128), torch.zeros(1 << 20, dtype=torch.uint8)
    c.k = c.k.transpose(1, 2)
    with pytest.raises(AssertionError):
        ngc.ngc_decode_attn(c, 0, q, 0.1, 0, out, ws, stream=0)
    c = _cache()
    c.k = c.k[0]
    with pytest.raises(ValueError):
        ngc.ngc_decode_attn(c, 0, q, 0.1, 0, out, ws, stream=0)
    c = _cache()
    for bad in (dict(q="x"), dict(q=3.0)):
        with pytest.raises(AttributeError):
            ngc.ngc_decode_attn(c, 0, bad["q"], 0.1, 0, out, ws, stream=0)
    with pytest.raises(TypeError):
        ngc.ngc_decode_attn(c, "0", q, 0.1, 0, out, ws, stream=0)
    with pytest.raises(TypeError):
        ngc.ngc_decode_attn(c, 0, q, "0.1", 0, out, ws, stream=0)
    with pytest.raises(AttributeError):
        ngc.ngc_decode_attn(c, 0, q, 0.1, 0, out, None, stream=0)
    front = ngc._front()
    with pytest.raises(TypeError):
        front.decode_attn(c, 0)
    with pytest.raises(RuntimeError):
        front.open("/nonexistent/libngc.so")


def test_a_forked_child_asks_torch_for_the_stream_again(monkeypatch):
    import os
    from paper_2604_18002_amd import binding
    monkeypatch.setattr(binding, "_current_raw_stream", lambda: 0)
    pid = os.fork()
    if pid == 0:
        os._exit(0 if binding._current_raw_stream is None else 1)
    assert os.waitpid(pid, 0)[1] == 0 and binding._current_raw_stream is not None


def test_arguments_of_a_wrong_type_raise_what_ctypes_raises():
    c = _cache()
    q, out, ws = torch.zeros(3, 12, 128, dtype=torch.bfloat16), torch.zeros(3, 12, 128), torch.zeros(1 << 20, dtype=torch.uint8)
    for layer, scale, hint in (("0", 0.1, 0), (0.0, 0.1, 0), (0, "0.1", 0), (0, None, 0), (0, 0.1, [1]), (C.c_char(b"0"), 0.1, 0)):
        with pytest.raises(C.ArgumentError):
            ngc.ngc_decode_attn(c, layer, q, scale, hint, out, ws, stream=0)
    x, keep = torch.zeros(2, 3, 2, 64), torch.zeros(2, 3, 2, dtype=torch.int32)
    kept = torch.zeros(2, 3, 2, 8, dtype=torch.int32)

    class Other(C.Structure):
        _fields_ = [("bytes", C.c_char * C.sizeof(ngc.ngc_evict_params))]
    for params in (Other(), bytearray(C.sizeof(Other)), bytes(C.sizeof(Other)), None):
        with pytest.raises((C.ArgumentError, TypeError)):
            ngc.ngc_evict(c, 0, x, keep, params, 8, kept, None, None, ws, stream=0)

    class Params(ngc.ngc_evict_params):
        pass
    assert _code(ngc.ngc_evict, c, 0, x, keep, Params(block=0), 8, kept, None, None, ws) == ngc.NGC_EINVAL
    # numbers that ctypes takes: its own, and whatever has __index__ or __float__
    for layer in (C.c_int32(2), torch.tensor(2), True + 1):
        assert _code(ngc.ngc_decode_attn, c, layer, q, C.c_float(0.1), 0, out, ws) == ngc.NGC_EINVAL
    assert _code(ngc.ngc_decode_attn, c, 0, q, C.c_float(float("nan")), 0, out, ws) == ngc.NGC_EINVAL


def test_a_cache_with_a_view_of_its_own_is_asked_for_it(monkeypatch):
    q, out, ws = torch.zeros(3, 12, 128, dtype=torch.bfloat16), torch.zeros(3, 12, 128), torch.zeros(1 << 20, dtype=torch.uint8)
    asked = []

    class Narrow(ngc.Cache):
        def view(self):
            asked.append(1)
            v = ngc.Cache.view(self)
            v.D = 96                                         # a head size the library refuses
            return v
    c = _cache()
    c = Narrow(c.k, c.v, c.len, c.pos, c.Hq)
    assert _code(ngc.ngc_decode_attn, c, 0, q, 0.1, 0, out, ws) == ngc.NGC_EINVAL and asked == [1]

    c = _cache()                                             # overridden on the object, and on the class
    narrow = c.view()
    narrow.D = 96
    assert _code(ngc.ngc_decode_attn, c, 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_ENOSPC
    c.view = lambda: narrow
    assert _code(ngc.ngc_decode_attn, c, 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_EINVAL
    with monkeypatch.context() as m:
        m.setattr(ngc.Cache, "view", lambda self: narrow)
        assert _code(ngc.ngc_decode_attn, _cache(), 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_EINVAL

    class Inherits(ngc.Cache):                               # its own class, the binding's view
        pass
    c = _cache()
    assert _code(ngc.ngc_decode_attn, Inherits(c.k, c.v, c.len, c.pos, c.Hq), 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_ENOSPC

    class Plain:                                             # nothing but a view
        def __init__(self, v):
            self.view = lambda: v
    good = _cache()
    assert _code(ngc.ngc_decode_attn, Plain(good.view()), 2, q, 0.1, 0, out, ws) == ngc.NGC_EINVAL      # no layer 2
    assert _code(ngc.ngc_decode_attn, Plain(good.view()), 0, q, 0.1, 0, out, ws[:16]) == ngc.NGC_ENOSPC
    with pytest.raises(C.ArgumentError):
        ngc.ngc_decode_attn(Plain(ngc.make_params()), 0, q, 0.1, 0, out, ws, stream=0)
    with pytest.raises(ZeroDivisionError):
        ngc.ngc_decode_attn(type("Broken", (), {"view": lambda self: 1 // 0})(), 0, q, 0.1, 0, out, ws, stream=0)

    class NarrowPaged(ngc.PagedCache):
        def view(self):
            v = ngc.PagedCache.view(self)
            v.page_rows = 48
            return v
    pc = ngc.PagedCache.allocate(2, 3, 2, 12, 128, 32, 4, 40, device="cpu")
    pc = NarrowPaged(pc.k_pool, pc.v_pool, pc.pos_pool, pc.table, pc.len, pc.free_stack, pc.free_count, pc.Hq)
    assert _code(ngc.ngc_paged_decode_attn, pc, 0, q, 0.1, 0, out, ws) == ngc.NGC_EINVAL


def test_the_stream_is_found_without_the_private_way_to_it(monkeypatch):
    monkeypatch.setattr(ngc, "_current_raw_stream", None)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 77})())
    assert ngc._stream(None) == 77 and ngc._stream(None) == 77
