"""Key scores without normalisers as two launches: what the shares of a segment leave between them stands in the scores' own
entries below the segment's length.  The workspace gets status counts and nothing else, whoever's it is, and entries past
the length stay as they are; lengths on both sides of every change in the number of shares, per key and per block,
contiguous and paged.  Against fp64 attention on the CPU: 2e-4 relative plus 1e-9 (means of probabilities, each an
exponential of an fp32 sum)."""
import pytest

from test_gpu_score_shares import _ngc, _reference

pytestmark = pytest.mark.gpu


def test_scoring_a_view_with_the_workspace_of_the_whole_cache():
    import torch
    ngc = _ngc()
    L, B, H, G, D, cap = 28, 16, 2, 4, 64, 2100
    g = torch.Generator(device="cuda").manual_seed(1)
    k, v = (torch.randn(L, B, H, cap, D, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(L, B, 3, H * G, D, generator=g, device="cuda").to(torch.bfloat16)
    n = torch.full((L, B, H), cap, dtype=torch.int32, device="cuda")
    whole = ngc.Cache(k, v, n, None, H * G)
    ws = ngc.allocate_workspace(whole, 1)
    scores = torch.zeros(L, B, H, cap, device="cuda")
    q0 = q[3, :, 0].contiguous()
    out, want = torch.full((B, H * G, D), -7.0, device="cuda"), torch.zeros(B, H * G, D, device="cuda")
    print("[score-scratch] view", flush=True)
    ngc.ngc_decode_attn(whole, 3, q0, D ** -0.5, 0, want, ws)
    part = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    for block in (1, 32):
        for layers, seqs in ((1, B), (1, 2), (2, 4)):
            view = ngc.Cache(*(x[3:3 + layers, :seqs].contiguous() for x in (k, v, n)), None, H * G)
            got, alone = (torch.zeros(layers, seqs, H, cap, device="cuda") for _ in range(2))
            args = (q[3:3 + layers, :seqs].contiguous(), 3, D ** -0.5, 0, block)
            ngc.ngc_score_keys(view, -1, *args, got, ws)
            ngc.ngc_score_keys(view, -1, *args, alone, part)
            assert torch.equal(got, alone)            # (the workspace does not choose the route either)
            tickets = ws[ngc.STATUS_WORDS * 4:ngc.STATUS_WORDS * 4 + 12 * L * B * H]
            assert int(tickets.count_nonzero()) == 0
            ngc.ngc_decode_attn(whole, 3, q0, D ** -0.5, 0, out.fill_(-7.0), ws)
            assert torch.equal(out, want)


def _lengths_where_the_shares_change(R, cap, per_key):
    """The least length that so many shares' parts fit in, and one less."""
    at = [1, 127, 128, cap]
    for s in range(2, 33):
        words = 2 * R * s
        need = s * -(-words // 128) * 128 if per_key else next(n for n in range(words, 2 * words + 64) if words <= n - -(-n // 32))
        need = max(need, 128 * (s if per_key else s - 1) + (0 if per_key else 1))
        at += [need - 1, need]
    return [n for n in at if n <= cap]


@pytest.mark.parametrize("block", [1, 32, 48])
@pytest.mark.parametrize("w,G,D", [(1, 6, 128), (3, 7, 64), (5, 6, 128), (5, 12, 64), (4, 16, 128)])
@pytest.mark.parametrize("cap", [1023, 1024, 2047, 4160])
def test_shares_by_length(cap, w, G, D, block):
    import torch
    ngc = _ngc()
    H, scale = 2, D ** -0.5
    lens = _lengths_where_the_shares_change(w * G, cap, block != 32)
    lens = (lens * 2)[:len(lens) + len(lens) % 2]
    B, Hq = len(lens) // H, G * H
    lens = [lens[H * b:H * b + H] for b in range(B)]
    g = torch.Generator().manual_seed(cap + D)
    k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(B, w, Hq, D, generator=g).to(torch.bfloat16)
    n = torch.tensor(lens, dtype=torch.int32).view(1, B, H)
    k[torch.arange(cap) >= n[..., None]] = float("nan")
    c = ngc.Cache(k.cuda(), k.cuda(), n.cuda(), None, Hq)
    ws = ngc.allocate_workspace(c, 1)
    scores = torch.full((1, B, H, cap), -1.0, device="cuda")
    print(f"[score-scratch] cap={cap} w={w} G={G} D={D} block={block} segments={B * H}", flush=True)
    ngc.ngc_score_keys(c, 0, q.cuda(), w, scale, 0, block, scores, ws)
    got = scores.cpu().double()
    assert int(ws.count_nonzero()) == 0
    P = 32
    pages = -(-cap // P)
    pool = torch.full((B * H * pages, P, D), float("nan"), dtype=torch.bfloat16)
    table = torch.full((1, B, H, pages), -1, dtype=torch.int32)
    free = B * H * pages
    for b in range(B):
        for h in range(H):
            for j in range(-(-lens[b][h] // P)):
                free -= 1
                rows = k[0, b, h, j * P:(j + 1) * P]
                pool[free, :len(rows)] = rows
                table[0, b, h, j] = free
    pc = ngc.PagedCache(pool.cuda(), pool.cuda(), None, table.cuda(), n.cuda(), torch.zeros(1, dtype=torch.int32).cuda(),
                        torch.zeros(1, dtype=torch.int32).cuda(), Hq)
    paged = torch.full((1, B, H, pages * P), -1.0, device="cuda")
    ngc.ngc_paged_score_keys(pc, 0, q.cuda(), w, scale, 0, block, paged, ws)
    assert int(ws.count_nonzero()) == 0
    paged = paged.cpu().double()
    for b in range(B):
        psi, _ = _reference(k[0, b].double(), q[b].double(), lens[b], w, scale)
        for h in range(H):
            want = psi[h] if block == 1 else torch.stack([x.mean() for x in psi[h].split(block)])
            for x in (got[0, b, h], paged[0, b, h]):
                assert (x[:want.numel()] - want).abs().le(2e-4 * want + 1e-9).all(), (lens[b][h], block)
                assert (x[lens[b][h]:] == -1.0).all(), (lens[b][h], block)
