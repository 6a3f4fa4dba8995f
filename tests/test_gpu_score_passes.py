"""Key scores without normalisers: the two passes as launches that the workgroups of a segment share, at segments around a
share of 128 keys and shorter than their shares, and the single launches (eight waves, four) where the segments are many or
the capacity is small; with a whole workspace and with one of the status words alone.  Against fp64 attention on the CPU: 2e-4 relative plus 1e-9
(means of probabilities, each an exponential of an fp32 sum)."""
import pytest

from test_gpu_score_shares import _ngc, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [1, 32])
@pytest.mark.parametrize("w,G,D", [(1, 6, 128), (3, 7, 64), (5, 7, 128), (5, 12, 64), (4, 16, 128)])
@pytest.mark.parametrize("B,cap", [(1, 4200), (3, 513), (16, 640), (64, 513), (65, 513), (129, 130), (2, 100)])
def test_two_passes(B, cap, w, G, D, block):
    import torch
    ngc = _ngc()
    H, scale = 2, D ** -0.5
    g = torch.Generator().manual_seed(cap + D + B)
    edges = [n for n in (cap, 1, 127, 128, 129, 255, 257, 0, 384, 513, 2, 640, 4100) if n <= cap]
    lens = [[edges[(i * 5 + h * 3) % len(edges)] for h in range(H)] for i in range(B)]
    k = torch.randn(1, B, H, cap, D, generator=g).to(torch.bfloat16)
    q = torch.randn(B, w, G * H, D, generator=g).to(torch.bfloat16)
    n = torch.tensor(lens, dtype=torch.int32).view(1, B, H)
    dk = k.clone()
    dk[torch.arange(cap) >= n[..., None]] = float("nan")
    c = ngc.Cache(dk.cuda(), dk.cuda(), n.cuda(), None, G * H)
    full = ngc.allocate_workspace(c, 1)
    small = torch.zeros(64 * ((ngc.STATUS_WORDS * 4 + 63) // 64), dtype=torch.uint8, device="cuda")
    print(f"[score-passes] B={B} cap={cap} w={w} G={G} D={D} block={block}", flush=True)
    checked = [b for b in range(B) if b < 4 or b == B - 1]
    refs = {b: _reference(k[0, b].double(), q[b].double(), lens[b], w, scale)[0] for b in checked}
    for ws in (full, small):
        scores = torch.full((1, B, H, cap), float("nan"), device="cuda")
        ngc.ngc_score_keys(c, 0, q.cuda(), w, scale, 0, block, scores, ws)
        got = scores.cpu().double()
        assert all(v == 0 for v in ngc.read_status(ws))
        for b in checked:
            for h in range(H):
                want = refs[b][h]
                if block > 1 and want.numel():
                    want = torch.stack([x.mean() for x in want.split(block)])
                x = got[0, b, h, :want.numel()]
                assert (x - want).abs().le(2e-4 * want + 1e-9).all(), (b, h, (x - want).abs().max())
    # the tickets of decode attention are as they were
    assert int(full[:ngc.STATUS_WORDS * 4 + B * H * 12].count_nonzero()) == 0


def test_a_length_above_the_capacity_is_counted_once():
    import torch
    ngc = _ngc()
    c = ngc.Cache.allocate(1, 2, 2, 4, 64, 700)
    c.len.fill_(650)
    c.len[0, 1, 1] = 701
    ws = ngc.allocate_workspace(c, 1)
    scores = torch.zeros(1, 2, 2, 700, device="cuda")
    ngc.ngc_score_keys(c, -1, torch.zeros(1, 2, 3, 4, 64, dtype=torch.bfloat16, device="cuda"), 3, 0.125, 0, 1, scores, ws)
    assert sum(ngc.read_status(ws)) == 1
    assert torch.allclose(scores[0, 1, 1, :690], torch.full((690,), 1 / 699.0, device="cuda"), rtol=5e-3)
