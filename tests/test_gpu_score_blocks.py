"""Block means and head pooling of the key scores: blocks of one tile of 32 keys, of several, and of neither, pooled over heads
of different lengths (one empty), with the normalisers given and without, more items than a workgroup has threads.  Against
fp64 attention on the CPU: 2e-4 relative plus 1e-9 (means of probabilities, each an exponential of an fp32 sum)."""
import pytest

from test_gpu_score_shares import _ngc, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("pool", [True, False])
@pytest.mark.parametrize("block", [1, 7, 32, 33, 64, 96, 320])
@pytest.mark.parametrize("cap,D,Hq", [(97, 64, 9), (600, 128, 3)])
def test_block_means_and_pooling(cap, D, Hq, block, pool, given):
    import torch
    ngc = _ngc()
    L, B, H, w, scale = 2, 4, 3, 2, D ** -0.5
    g = torch.Generator().manual_seed(cap + block)
    edges = [n for n in (1, 31, 32, 33, 63, 64, 65, 95, 97, 257, 511, 513, 600) if n <= cap]
    lens = torch.tensor([edges[(i * 7) % len(edges)] for i in range(L * B * H)], dtype=torch.int32).view(L, B, H)
    lens[1, 2, 1] = 0
    k = torch.randn(L, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(L, B, w, Hq, D, generator=g).to(torch.bfloat16)
    refs = [[_reference(k[l, b].double(), q[l, b].double(), lens[l, b].tolist(), w, scale) for b in range(B)] for l in range(L)]
    lse = torch.stack([torch.stack([r[1] for r in row]) for row in refs]).float().cuda() if given else None
    dk = k.clone()
    dk[torch.arange(cap) >= lens[..., None]] = float("nan")
    c = ngc.Cache(dk.cuda(), dk.cuda(), lens.cuda(), None, Hq)
    ws = ngc.allocate_workspace(c, 1)
    scores = torch.full((L, B, H, cap), float("nan"), device="cuda")
    print(f"[score-blocks] cap={cap} D={D} block={block} pool={pool} given={given}", flush=True)
    ngc.ngc_score_keys(c, -1, q.cuda(), w, scale, ngc.SCORE_POOL_HEADS if pool else 0, block, scores, ws, lse_recent=lse)
    one = torch.full((L, B, H, cap), float("nan"), device="cuda")
    ngc.ngc_score_keys(c, 1, q[1].contiguous().cuda(), w, scale, ngc.SCORE_POOL_HEADS if pool else 0, block, one, ws,
                       lse_recent=None if lse is None else lse[1].contiguous())
    got, one = scores.cpu().double(), one.cpu().double()
    assert torch.isnan(one[0]).all()
    for l in range(L):
        for b in range(B):
            means = [torch.stack([x.mean() for x in p.split(block)]) if p.numel() else p for p in refs[l][b][0]]
            if pool:
                items = max(m.numel() for m in means)
                pooled = torch.stack([torch.stack([m[j] for m in means if m.numel() > j]).mean() for j in range(items)])
                means = [pooled[:m.numel()] for m in means]
            for h, want in enumerate(means):
                x = got[l, b, h, :want.numel()]
                assert (x - want).abs().le(2e-4 * want + 1e-9).all(), (l, b, h, (x - want).abs().max())
                if l == 1:
                    assert torch.equal(one[l, b, h, :want.numel()], x), (b, h)
    assert all(v == 0 for v in ngc.read_status(ws))


# sequences that share the pooling workgroups: one to a sequence, two (three would be a thread per item), one per 256 items
@pytest.mark.parametrize("B,H,cap", [(2049, 1, 300), (1100, 2, 700), (40, 3, 1030)])
def test_pooling_workgroups(B, H, cap):
    import torch
    ngc = _ngc()
    D, G, w = 64, 2, 1
    g = torch.Generator(device="cuda").manual_seed(cap)
    k = torch.randn(1, B, H, cap, D, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(B, w, H * G, D, generator=g, device="cuda").to(torch.bfloat16)
    n = torch.randint(0, cap + 1, (1, B, H), generator=g, device="cuda", dtype=torch.int32)
    n[0, 0] = cap
    n[0, 1] = 0
    c = ngc.Cache(k, k, n, None, H * G)
    ws = ngc.allocate_workspace(c, 1)
    alone, pooled = torch.zeros(1, B, H, cap, device="cuda"), torch.full((1, B, H, cap), -1.0, device="cuda")
    print(f"[score-blocks] pooling B={B} H={H} cap={cap}", flush=True)
    ngc.ngc_score_keys(c, 0, q, w, D ** -0.5, 0, 1, alone, ws)
    ngc.ngc_score_keys(c, 0, q, w, D ** -0.5, ngc.SCORE_POOL_HEADS, 1, pooled, ws)
    has = torch.arange(cap, device="cuda") < n[..., None]
    want = (alone.double() * has).sum(2, keepdim=True) / has.sum(2, keepdim=True).clamp(min=1)
    # up to H fp32 additions and a division
    assert (torch.where(has, (pooled.double() - want).abs(), 0.0) <= 1e-6 * want + 1e-30).all()
    assert (pooled[~has] == -1.0).all()
