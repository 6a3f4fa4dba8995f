"""Decode attention at the edges of its tiles and rounds: lengths around one row, one 32-row tile, one round of four tiles
per workgroup and the counts where the number of workgroups per segment changes, every unused row of the cache holding
NaN (a wave asks for its first tile before it knows the length, and the appended row is put into its tile from the
call's arguments, so none of these rows may reach the result), both head sizes, every entry point.

Against fp64 attention on the CPU, 1e-4 absolute: the probabilities enter the second product with 2^-16 relative error
against values of at most ~5, the rest is fp32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-4
LENGTHS = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 161, 255, 256, 257, 383, 385, 511, 512, 513, 700, 1023, 1025]


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _reference(q, k, v, n, scale):
    """q [Hq, D], k, v [H, N, D] (fp64), n [H] -> [Hq, D], lse [Hq]"""
    import torch
    H, N, D = k.shape
    out, lse = [], []
    for h in range(H):
        s = q.view(H, -1, D)[h] @ k[h, :n[h]].t() * scale
        out.append(torch.softmax(s, -1) @ v[h, :n[h]])
        lse.append(torch.logsumexp(s, -1))
    return torch.cat(out), torch.cat(lse)


@pytest.mark.parametrize("B", [1, 6, 40])         # 2, 12, 80 segments: up to 64, 21 and 3 workgroups a segment
@pytest.mark.parametrize("D,Hq", [(64, 8), (128, 12)])
def test_lengths_around_tiles_and_rounds_with_nan_beyond_them(B, D, Hq):
    import torch
    ngc = _ngc()
    H, cap, scale = 2, 1040, D ** -0.5
    g = torch.Generator().manual_seed(B * 1000 + D)
    lens = [LENGTHS[(i * 7 + B) % len(LENGTHS)] for i in range(B * H)]
    if B == 1:
        groups = [LENGTHS[i:i + 2] for i in range(0, len(LENGTHS), 2)]
    else:
        groups = [lens]
    for lens in groups:
        n = torch.tensor(lens, dtype=torch.int32).view(1, B, H)
        k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
        v = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
        q = torch.randn(B, Hq, D, generator=g).to(torch.bfloat16)
        row = torch.arange(cap)
        for grow in (False, True):
            used = (n - 1 if grow else n)                     # rows in the cache before the call
            unused = row[None, None, None] >= used[..., None]
            dk, dv = k.clone(), v.clone()
            dk[unused], dv[unused] = float("nan"), float("nan")
            for hint in (0, int(n.max()), 4 * int(n.max())):
                c = ngc.Cache(dk.cuda(), dv.cuda(), used.cuda().contiguous(), None, Hq)
                ws = ngc.allocate_workspace(c, 1)
                out, lse = torch.zeros(B, Hq, D, device="cuda"), torch.zeros(B, Hq, device="cuda")
                print(f"[decode-edges] B={B} D={D} grow={grow} hint={hint} n={lens[:4]}", flush=True)
                if grow:
                    at = (n[0].long() - 1)[..., None, None].expand(B, H, 1, D)
                    kn, vn = k[0].gather(2, at)[:, :, 0], v[0].gather(2, at)[:, :, 0]
                    ngc.ngc_decode_step(c, 0, kn.cuda().contiguous(), vn.cuda().contiguous(), None, q.cuda(), scale,
                                        hint, out, ws, lse_out=lse)
                else:
                    ngc.ngc_decode_attn(c, 0, q.cuda(), scale, hint, out, ws, lse_out=lse)
                    out2 = torch.zeros_like(out)
                    ngc.ngc_decode_attn_static(c, 0, q.cuda(), scale, hint, out2)
                    assert torch.equal(out, out2)
                assert torch.equal(c.len.cpu(), n)
                assert ngc.read_status(ws)[:4] == [0, 0, 0, 0]
                got, got_lse = out.cpu().double(), lse.cpu().double()
                for b in range(B):
                    want, want_lse = _reference(q[b].double(), k[0, b].double(), v[0, b].double(), n[0, b].tolist(), scale)
                    assert (got[b] - want).abs().max() <= TOL, (b, lens[2 * b:2 * b + 2])
                    assert (got_lse[b] - want_lse).abs().max() <= 2e-5, (b, lens[2 * b:2 * b + 2])
                if grow:
                    hk, hv = c.k.cpu()[0], c.v.cpu()[0]
                    assert torch.equal(hk.gather(2, at)[:, :, 0], kn) and torch.equal(hv.gather(2, at)[:, :, 0], vn)


@pytest.mark.parametrize("page", [32, 128])
def test_paged_lengths_with_nan_beyond_them_and_stale_table_entries(page):
    import torch
    ngc = _ngc()
    B, H, Hq, D, scale = 6, 2, 12, 128, 128 ** -0.5
    g = torch.Generator().manual_seed(page)
    lens = [LENGTHS[(i * 5) % len(LENGTHS)] for i in range(B * H)]
    n = torch.tensor(lens, dtype=torch.int32).view(1, B, H)
    max_pages = 1040 // page + 2
    num_pages = B * H * max_pages
    order = torch.randperm(num_pages, generator=g).to(torch.int32)
    table = torch.where(torch.rand(1, B, H, max_pages, generator=g) < 0.5, torch.tensor(-7), torch.tensor(1 << 30)).to(torch.int32)
    kp = torch.full((num_pages, page, D), float("nan"), dtype=torch.bfloat16)
    vp = kp.clone()
    k = torch.randn(B, H, 1040, D, generator=g).to(torch.bfloat16)
    v = torch.randn(B, H, 1040, D, generator=g).to(torch.bfloat16)
    used = 0
    for b in range(B):
        for h in range(H):
            m = int(n[0, b, h])
            for j in range((m + page - 1) // page):
                p = int(order[used])
                used += 1
                table[0, b, h, j] = p
                rows = min(page, m - j * page)
                kp[p, :rows], vp[p, :rows] = k[b, h, j * page:j * page + rows], v[b, h, j * page:j * page + rows]
    q = torch.randn(B, Hq, D, generator=g).to(torch.bfloat16)
    pc = ngc.PagedCache(kp.cuda(), vp.cuda(), None, table.cuda(), n.cuda(), torch.zeros(num_pages, dtype=torch.int32).cuda(),
                        torch.zeros(1, dtype=torch.int32).cuda(), Hq)
    ws = ngc.allocate_paged_workspace(pc)
    for hint in (0, 600, 1040):
        out, lse = torch.zeros(B, Hq, D, device="cuda"), torch.zeros(B, Hq, device="cuda")
        print(f"[decode-edges] paged page={page} hint={hint}", flush=True)
        ngc.ngc_paged_decode_attn(pc, 0, q.cuda(), scale, hint, out, ws, lse_out=lse)
        for b in range(B):
            want, want_lse = _reference(q[b].double(), k[b].double(), v[b].double(), n[0, b].tolist(), scale)
            assert (out.cpu().double()[b] - want).abs().max() <= TOL, b
            assert (lse.cpu().double()[b] - want_lse).abs().max() <= 2e-5, b


def test_split_rule_stays_inside_the_workspace_it_promises():
    """Whatever the length hint, the partials of a launch fit the workspace (a launch that finds less quietly takes fewer
    workgroups): results with the promised size and with a far larger one are the same bits."""
    import torch
    ngc = _ngc()
    B, H, Hq, D, cap = 3, 2, 32, 128, 3000
    g = torch.Generator(device="cuda").manual_seed(5)
    c = ngc.Cache(torch.randn(1, B, H, cap, D, generator=g, device="cuda").to(torch.bfloat16),
                  torch.randn(1, B, H, cap, D, generator=g, device="cuda").to(torch.bfloat16),
                  torch.full((1, B, H), 2900, dtype=torch.int32, device="cuda"), None, Hq)
    q = torch.randn(B, Hq, D, generator=g, device="cuda").to(torch.bfloat16)
    ws = ngc.allocate_workspace(c, 1)
    big = torch.zeros(ws.numel() + (16 << 20), dtype=torch.uint8, device="cuda")
    for hint in [0] + list(range(100, 3001, 100)):
        a, b = torch.zeros(B, Hq, D, device="cuda"), torch.zeros(B, Hq, D, device="cuda")
        ngc.ngc_decode_attn(c, 0, q, D ** -0.5, hint, a, ws)
        ngc.ngc_decode_attn(c, 0, q, D ** -0.5, hint, b, big)
        assert torch.equal(a, b), hint


@pytest.mark.parametrize("D,Hq", [(64, 8), (128, 12)])
# the first tile before the length, after it (three times), and before it again
@pytest.mark.parametrize("B,hint", [(128, 65), (128, 64), (129, 0), (129, 128), (129, 129)])
def test_first_tile_before_and_after_the_length(B, hint, D, Hq):
    """256 segments of one workgroup each are the most for which a wave asks for its first tile before it knows the length
    whatever the caller knows, and only if the longest may have more than two tiles; beyond, the caller has to know that the
    longest has more than 128 rows.  Both sides of each limit, empty and full segments among them,
    NaN in every unused row, contiguous (with and without the append) and paged."""
    import torch
    ngc = _ngc()
    H, scale = 2, D ** -0.5
    cap = hint or 160
    g = torch.Generator().manual_seed(B + hint + D)
    edges = [x for x in (0, 1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 159, 160, 255) if x <= cap] + [cap]
    n = torch.tensor([edges[(i * 5) % len(edges)] for i in range(B * H)], dtype=torch.int32).view(1, B, H)
    k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    v = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(B, Hq, D, generator=g).to(torch.bfloat16)
    kn, vn = (torch.randn(B, H, D, generator=g).to(torch.bfloat16) for _ in range(2))
    unused = torch.arange(cap)[None, None, None] >= n[..., None]
    k[unused], v[unused] = float("nan"), float("nan")

    def check(out, lse, kk, vv, m, what):
        for b in range(B):
            for h in range(H):
                rows, got = int(m[0, b, h]), out[b].view(H, -1, D)[h].cpu().double()
                if rows == 0:
                    assert (got == 0).all() and torch.isneginf(lse[b].view(H, -1)[h]).all(), (what, b, h)
                    continue
                s = q[b].double().view(H, -1, D)[h] @ kk[0, b, h, :rows].double().t() * scale
                assert (got - torch.softmax(s, -1) @ vv[0, b, h, :rows].double()).abs().max() <= TOL, (what, b, h, rows)
                assert (lse[b].view(H, -1)[h].cpu().double() - torch.logsumexp(s, -1)).abs().max() <= 2e-5, (what, b, h, rows)

    out, lse = torch.zeros(B, Hq, D, device="cuda"), torch.zeros(B, Hq, device="cuda")
    c = ngc.Cache(k.cuda(), v.cuda(), n.cuda(), None, Hq)
    ws = ngc.allocate_workspace(c, 1)
    print(f"[decode-edges] early B={B} hint={hint} D={D}", flush=True)
    ngc.ngc_decode_attn(c, 0, q.cuda(), scale, hint, out, ws, lse_out=lse)
    check(out, lse, k, v, n, "attn")
    ngc.ngc_decode_step(c, 0, kn.cuda(), vn.cuda(), None, q.cuda(), scale, hint, out, ws, lse_out=lse)
    grown = torch.minimum(n + 1, torch.tensor(cap, dtype=torch.int32))
    assert torch.equal(c.len.cpu(), grown)
    k2, v2 = k.clone(), v.clone()
    for b in range(B):
        for h in range(H):
            if n[0, b, h] < cap:
                k2[0, b, h, n[0, b, h]], v2[0, b, h, n[0, b, h]] = kn[b, h], vn[b, h]
    check(out, lse, k2, v2, grown, "step")
    assert ngc.read_status(ws)[:4] == [0, 0, int((n == 0).sum()), int((n == cap).sum())]

    pages = (cap + 31) // 32
    table = torch.randperm(B * H * pages, generator=g).to(torch.int32).view(1, B, H, pages)
    pad = torch.full((1, B, H, pages * 32, D), float("nan"), dtype=torch.bfloat16)
    pools = []
    for x in (k, v):
        p = pad.clone()
        p[:, :, :, :cap] = x
        pool = torch.empty(B * H * pages, 32, D, dtype=torch.bfloat16)
        pool[table.flatten().long()] = p.view(-1, 32, D)
        pools.append(pool.cuda())
    stale = torch.arange(pages)[None, None, None] * 32 >= n[..., None]
    table[stale] = 1 << 30
    pc = ngc.PagedCache(pools[0], pools[1], None, table.cuda(), n.cuda(), torch.zeros(B * H * pages, dtype=torch.int32).cuda(),
                        torch.zeros(1, dtype=torch.int32).cuda(), Hq)
    print(f"[decode-edges] early paged B={B} hint={hint} D={D}", flush=True)
    ngc.ngc_paged_decode_attn(pc, 0, q.cuda(), scale, hint, out, ngc.allocate_paged_workspace(pc), lse_out=lse)
    check(out, lse, k, v, n, "paged")


@pytest.mark.parametrize("lost", ["a wave", "first tiles", "a workgroup", "all but a row"])
@pytest.mark.parametrize("B", [2, 130])           # several workgroups a segment, one
@pytest.mark.parametrize("D,Hq", [(64, 8), (128, 12)])
def test_rows_that_score_minus_infinity(B, D, Hq, lost):
    """Rows that score -inf for every query add nothing, whether they are all that one wave of four sees, the first that every
    wave sees, all that a workgroup of a shared segment sees, or nearly all there are: output and log-sum-exp are those of the
    other rows (tolerances as above).  A row of NaN is not hidden by them."""
    import torch
    ngc = _ngc()
    H, cap, scale = 2, 500, D ** -0.5
    g = torch.Generator().manual_seed(B + D)
    n = torch.full((1, B, H), cap, dtype=torch.int32)
    k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    v = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(B, Hq, D, generator=g).to(torch.bfloat16)
    q[..., 0] = 1
    tile = torch.arange(cap) // 32                    # tile t: wave t % 4 of workgroup t / 4 modulo the workgroups
    gone = {"a wave": tile % 4 == 1, "first tiles": tile < 12, "a workgroup": tile // 4 == 1,
            "all but a row": torch.arange(cap) != 77}[lost]
    s = q.double().view(B, H, -1, D) @ k[0][:, :, ~gone].double().transpose(-1, -2) * scale
    want_lse, want = torch.logsumexp(s, -1), torch.softmax(s, -1) @ v[0][:, :, ~gone].double()
    k[..., gone, 0] = float("-inf")
    for nan in (False, True):
        if nan:
            k[:, -1, :, 40, 0] = float("nan")
        out, lse = torch.zeros(B, Hq, D, device="cuda"), torch.zeros(B, Hq, device="cuda")
        c = ngc.Cache(k.cuda(), v.cuda(), n.cuda(), None, Hq)
        ws = ngc.allocate_workspace(c, 1)
        print(f"[decode-edges] -inf {lost} B={B} D={D} nan={nan}", flush=True)
        ngc.ngc_decode_attn(c, 0, q.cuda(), scale, cap, out, ws, lse_out=lse)
        got, got_lse = out.cpu().double().view_as(want), lse.cpu().double().view_as(want_lse)
        m = B - 1 if nan else B
        assert (got_lse[:m] - want_lse[:m]).abs().max() <= 2e-5
        assert (got[:m] - want[:m]).abs().max() <= TOL
        if nan:
            assert torch.isnan(got[-1]).all() and torch.isnan(got_lse[-1]).all()
