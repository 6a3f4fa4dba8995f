"""Replay attention on both sides of the length up to which the workgroups make their own key lists (2048 positions; 1536 for
many workgroups that share lists), and at the edges of a list: passes of 256 positions, lists that fill their tile or the whole buffer, query tiles without any key,
last tiles in which only the first wave has queries, death positions far outside the trajectory."""
import pytest

from test_gpu_replay_edges import _check

pytestmark = pytest.mark.gpu


def _deaths(T, kind, rows, seed):
    import torch
    g = torch.Generator().manual_seed(seed)
    if kind == "any":
        return torch.randint(1, 2 * T + 2, (rows, T), generator=g).to(torch.int32)
    if kind == "never":
        return torch.full((rows, T), 2 ** 31 - 1, dtype=torch.int32)
    if kind == "at once":                                     # nobody sees anything
        return torch.arange(T, dtype=torch.int32).repeat(rows, 1)
    d = torch.randint(-2 ** 31, 2 ** 31 - 1, (rows, T), generator=g)      # all or nothing, the halves of a list
    d[:, ::3] = 70000
    return d.to(torch.int32)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T", [255, 256, 257, 513, 1024, 1027, 1793, 2047, 2048, 2049, 2177])
def test_lengths_around_passes_and_the_limit(T, D):
    _check(1, T, 4, 2, D, _deaths(T, "any", 2, T).view(1, 2, T).cuda(), T)


@pytest.mark.parametrize("T", [130, 640, 2048, 2080])
@pytest.mark.parametrize("kind", ["never", "at once", "extremes"])
def test_full_empty_and_extreme_lists(T, kind):
    _check(2, T, 3, 1, 64, _deaths(T, kind, 2, T).cuda(), T)


# 13 tiles x 4 heads: 79 trajectories are 4108 workgroups, on the list kernel's route; alone each makes its own lists
@pytest.mark.parametrize("T,B,Hkv", [(1536, 88, 2), (1537, 78, 2), (1537, 79, 2), (1600, 79, 1), (1600, 80, 4)])
def test_many_trajectories_give_what_each_gives_alone(T, B, Hkv):
    import torch
    from paper_2604_18002_amd import binding as ngc
    Hq, D = 4, 64
    g = torch.Generator("cuda").manual_seed(B)
    q = torch.randn(B, T, Hq, D, generator=g, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn(B, T, Hkv, D, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    death = _deaths(T, "any", B * Hkv, B).view(B, Hkv, T).cuda()
    ws = torch.zeros(ngc.ngc_replay_workspace_bytes(B, T, Hkv), dtype=torch.uint8, device="cuda")
    out, one = torch.zeros(B, T, Hq, D, device="cuda"), torch.zeros(1, T, Hq, D, device="cuda")
    print(f"[replay-routes] T={T} B={B} {Hq}/{Hkv}", flush=True)
    ngc.ngc_replay_attn(q, k, v, death, B, T, Hq, Hkv, D, True, D ** -0.5, out, ws)
    for b in (0, B // 2, B - 1):
        part = [x[b:b + 1].contiguous() for x in (q, k, v, death)]
        ngc.ngc_replay_attn(*part, 1, T, Hq, Hkv, D, True, D ** -0.5, one, ws)
        assert torch.equal(out[b], one[0]), b
