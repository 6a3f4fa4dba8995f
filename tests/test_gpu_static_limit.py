"""Which calls the no-workspace decode entry point takes, for the one head geometry that can outgrow its array (16 query heads
per KV head, D = 128): the rule is on sizes and stands whatever split is launched; what is taken returns the bits of the
entry point with a workspace."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


def _taken(nseg, rows):
    s = min(256 // nseg, int((80.0 * 2 * 256 * rows * 1e-6) ** 0.5), (rows + 31) // 32 // 4, 64)
    up = lambda x: (x + 255) // 256 * 256
    return s <= 1 or 4096 + up(nseg * s * 16 * 128 * 4) + up(nseg * s * 16 * 2 * 4) <= 2 << 20


@pytest.mark.parametrize("B,cap,hint", [(16, 3000, 0), (16, 1500, 0), (16, 9000, 0), (16, 9000, 1500), (32, 525, 0),
                                        (64, 1500, 0), (128, 525, 0), (5, 12000, 0), (1, 4000, 0)])
def test_taken_or_refused(B, cap, hint):
    import torch
    from paper_2604_18002_amd import binding as ngc
    lib = ngc.load_library()
    g = torch.Generator(device="cuda").manual_seed(cap + B)
    k = torch.randn(1, B, 1, cap, 128, generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn(1, B, 1, cap, 128, generator=g, device="cuda", dtype=torch.bfloat16)
    n = torch.randint(cap // 2, cap + 1, (1, B, 1), generator=g, device="cuda", dtype=torch.int32)
    q = torch.randn(B, 16, 128, generator=g, device="cuda", dtype=torch.bfloat16)
    c = ngc.Cache(k, v, n, None, 16)
    ws = ngc.allocate_workspace(c, 1)
    want, got = torch.zeros(B, 16, 128, device="cuda"), torch.zeros(B, 16, 128, device="cuda")
    st = ngc.ngc_cache(k.data_ptr(), v.data_ptr(), n.data_ptr(), None, 1, B, 1, 16, 128, cap)
    print(f"[static-limit] B={B} cap={cap} hint={hint}", flush=True)
    rc = lib.ngc_decode_attn_static(C.byref(st), 0, q.data_ptr(), 0.08, hint, got.data_ptr(), None, None,
                                    torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == (0 if _taken(B, hint or cap) else ngc.NGC_ENOSPC)
    ngc.ngc_decode_attn(c, 0, q, 0.08, hint, want, ws)
    if rc == 0:
        assert torch.equal(got, want)
    ref = [torch.softmax(q[b].double() @ k[0, b, 0, :n[0, b, 0]].double().t() * 0.08, -1)
           @ v[0, b, 0, :n[0, b, 0]].double() for b in range(B)]
    assert (want.double() - torch.stack(ref)).abs().max() <= 2e-3
