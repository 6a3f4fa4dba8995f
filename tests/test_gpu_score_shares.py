"""Key scores with the normalisers given, where a segment is shared by several workgroups: lengths around a 32-row tile and a
round of four tiles, more workgroups than rounds, both head sizes, contiguous and paged, per key and per block.  Against
fp64 attention on the CPU: 2e-4 relative plus 1e-9 (means of probabilities, each an exponential of an fp32 sum)."""
import pytest

pytestmark = pytest.mark.gpu


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _reference(k, q, n, w, scale):
    """k [H, N, D], q [w, Hq, D] (fp64), n [H] -> list of psi [n] per head, lse [w, Hq]"""
    import torch
    H, G = k.shape[0], q.shape[1] // k.shape[0]
    psi, lse = [], torch.full((w, q.shape[1]), float("-inf"), dtype=torch.float64)
    for h in range(H):
        acc = torch.zeros(n[h], dtype=torch.float64)
        for j in range(w):
            vis = n[h] - w + j + 1
            if vis <= 0:
                continue
            s = q[j, h * G:(h + 1) * G] @ k[h, :vis].t() * scale
            lse[j, h * G:(h + 1) * G] = torch.logsumexp(s, -1)
            acc[:vis] += torch.softmax(s, -1).sum(0)
        psi.append(acc / (w * G))
    return psi, lse


@pytest.mark.parametrize("block", [1, 32])
@pytest.mark.parametrize("D,Hq", [(64, 8), (128, 12)])
@pytest.mark.parametrize("B,cap", [(1, 1030), (3, 700), (48, 300)])
def test_shared_segments(B, cap, D, Hq, block):
    import torch
    ngc = _ngc()
    H, w, scale = 2, 3, D ** -0.5
    g = torch.Generator().manual_seed(cap + D)
    pool = [n for n in (3, 31, 32, 33, 127, 128, 129, 255, 257, 300, 511, 513, 700, 1023, 1025, 1030) if n <= cap]
    lens = [[pool[(i * 5 + h * 3 + B) % len(pool)] for h in range(H)] for i in range(B)]
    k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(B, w, Hq, D, generator=g).to(torch.bfloat16)
    refs = [_reference(k[0, b].double(), q[b].double(), lens[b], w, scale) for b in range(B)]
    lse = torch.stack([r[1] for r in refs]).float()
    row = torch.arange(cap)
    n = torch.tensor(lens, dtype=torch.int32).view(1, B, H)
    dk = k.clone()
    dk[row[None, None, None] >= n[..., None]] = float("nan")
    c = ngc.Cache(dk.cuda(), dk.cuda(), n.cuda(), None, Hq)
    ws = ngc.allocate_workspace(c, 1)
    scores = torch.full((1, B, H, cap), -1.0, device="cuda")
    print(f"[score-shares] B={B} cap={cap} D={D} block={block}", flush=True)
    ngc.ngc_score_keys(c, 0, q.cuda(), w, scale, 0, block, scores, ws, lse_recent=lse.cuda())
    # the same rows over pages in reverse order
    P = 32
    pages = (cap + P - 1) // P
    kp = torch.full((B * H * pages, P, D), float("nan"), dtype=torch.bfloat16)
    table = torch.full((1, B, H, pages), -1, dtype=torch.int32)
    for b in range(B):
        for h in range(H):
            for j in range((lens[b][h] + P - 1) // P):
                at = (b * H + h + 1) * pages - 1 - j
                table[0, b, h, j] = at
                rows = dk[0, b, h, j * P:(j + 1) * P]
                kp[at, :rows.shape[0]] = rows
    pc = ngc.PagedCache(kp.cuda(), kp.cuda(), None, table.cuda(), n.cuda(), torch.zeros(1, dtype=torch.int32).cuda(),
                        torch.zeros(1, dtype=torch.int32).cuda(), Hq)
    pws = ngc.allocate_paged_workspace(pc)
    paged = torch.full((1, B, H, pages * P), -1.0, device="cuda")
    ngc.ngc_paged_score_keys(pc, 0, q.cuda(), w, scale, 0, block, paged, pws, lse_recent=lse.cuda())
    for got in (scores.cpu().double(), paged.cpu().double()):
        for b in range(B):
            for h in range(H):
                m, want = lens[b][h], refs[b][0][h]
                if block > 1:
                    want = torch.stack([x.mean() for x in want.split(block)])
                x = got[0, b, h, :want.numel()]
                assert (x - want).abs().le(2e-4 * want + 1e-9).all(), (b, h, m, (x - want).abs().max())
                if block == 1:
                    assert (got[0, b, h, m:] == -1.0).all()
    assert all(v == 0 for v in ngc.read_status(ws))


@pytest.mark.parametrize("B,cap,D,w", [(257, 2048, 64, 4), (768, 2050, 64, 4), (769, 2048, 64, 4), (257, 2048, 128, 4),
                                       (320, 2050, 128, 9), (321, 2048, 128, 4), (512, 2048, 128, 9), (513, 2048, 128, 9),
                                       (768, 2050, 128, 9), (769, 2048, 128, 9)])
def test_second_workgroup_of_long_segments(B, cap, D, w):
    """More segments than CUs twice over: at D = 128 those of 2048 rows and more are shared by two workgroups (up to 640
    segments), shorter ones are not; the last rows are not seen by all queries.  Either side of that, and of the numbers of
    segments between which launches with two query tiles keep to three workgroups a CU.  Only a few segments are compared."""
    import torch
    ngc = _ngc()
    H, Hq = 2, 4
    scale = D ** -0.5
    g = torch.Generator().manual_seed(B + cap)
    lens = torch.full((1, B, H), 5, dtype=torch.int32)
    rows = {0: (2048, 2047), 1: (cap, 33), B - 1: (2045, 2048)}
    k = torch.zeros(1, B, H, cap, D, dtype=torch.bfloat16, device="cuda")
    q = torch.randn(B, w, Hq, D, generator=g).to(torch.bfloat16)
    lse = torch.zeros(B, w, Hq)
    refs = {}
    for b, n in rows.items():
        kb = torch.randn(H, cap, D, generator=g).to(torch.bfloat16)
        refs[b], e = _reference(kb.double(), q[b].double(), n, w, scale)
        lse[b] = e.float()
        for h in range(H):
            lens[0, b, h] = n[h]
            kb[h, n[h]:] = float("nan")
        k[0, b] = kb.cuda()
    c = ngc.Cache(k, k, lens.cuda(), None, Hq)
    ws = ngc.allocate_workspace(c, 1)
    scores = torch.full((1, B, H, cap), -1.0, device="cuda")
    print(f"[score-shares] second workgroup B={B} cap={cap}", flush=True)
    ngc.ngc_score_keys(c, 0, q.cuda(), w, scale, 0, 1, scores, ws, lse_recent=lse.cuda())
    got = scores.cpu().double()[0]
    for b, n in rows.items():
        for h in range(H):
            want = refs[b][h]
            assert torch.all((got[b, h, :n[h]] - want).abs() <= 2e-4 * want.abs() + 1e-9), (b, h)
            assert torch.all(got[b, h, n[h]:] == -1.0)
    assert torch.all(got[2:B - 1, :, 5:] == -1.0) and torch.isfinite(got).all()
