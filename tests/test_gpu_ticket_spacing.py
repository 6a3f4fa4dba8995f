"""Split decode launches and where their tickets lie: as far apart as the words of the workspace (one per segment of the
cache) or of the fixed array allow, up to 32 words.  Caches of one layer (next to each other), a few (between), more than
32 (a whole line apart), segment counts that do not divide the words.

The entry point without a workspace splits the same way and returns the same bits; a cache of one layer holding the same rows
may be split another way (the split follows the spacing).  1e-4 absolute, there and against fp64 attention on the CPU: the
probabilities enter the second product with 2^-16 relative error against values of at most ~5, the rest is fp32."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,B,H,D", [(1, 3, 2, 64), (2, 5, 3, 64), (7, 9, 1, 64), (28, 16, 2, 64), (33, 2, 2, 64), (40, 21, 3, 64),
                                     (5, 8, 2, 128), (28, 24, 2, 128)])
def test_layers_agree_with_caches_of_one_layer(L, B, H, D):
    import torch
    from paper_2604_18002_amd import binding as ngc
    ngc.load_library()
    G, cap = 4, 660
    g = torch.Generator(device="cuda").manual_seed(L * 100 + B)
    k, v = (torch.randn(L, B, H, cap, D, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(L, B, H * G, D, generator=g, device="cuda").to(torch.bfloat16)
    n = torch.randint(1, cap + 1, (L, B, H), generator=g, device="cuda", dtype=torch.int32)
    scale = D ** -0.5
    cache = ngc.Cache(k, v, n, None, H * G)
    ws = ngc.allocate_workspace(cache, 1)
    for again in range(2):                        # the second time over tickets that the first has put back to zero
        for l in range(L):
            print(f"[tickets] L={L} B={B} H={H} layer={l} again={again}", flush=True)
            got, static, want = (torch.zeros(B, H * G, D, device="cuda") for _ in range(3))
            ngc.ngc_decode_attn(cache, l, q[l], scale, 0, got, ws)
            ngc.ngc_decode_attn_static(cache, l, q[l], scale, 0, static)
            one = ngc.Cache(k[l:l + 1], v[l:l + 1], n[l:l + 1], None, H * G)
            ngc.ngc_decode_attn(one, 0, q[l], scale, 0, want, ngc.allocate_workspace(one, 1))
            assert torch.equal(static, got)
            assert (got - want).abs().max() <= 1e-4
    tickets = ws[ngc.STATUS_WORDS * 4:ngc.STATUS_WORDS * 4 + 12 * L * B * H].view(torch.int32)
    assert int(tickets.abs().sum()) == 0 and all(x == 0 for x in ngc.read_status(ws))
    for b in range(B):
        for h in range(H):
            m = int(n[L - 1, b, h])
            s = q[L - 1, b, h * G:(h + 1) * G].cpu().double() @ k[L - 1, b, h, :m].cpu().double().t() * scale
            ref = torch.softmax(s, -1) @ v[L - 1, b, h, :m].cpu().double()
            assert (got[b, h * G:(h + 1) * G].cpu().double() - ref).abs().max() <= 1e-4, (b, h)
