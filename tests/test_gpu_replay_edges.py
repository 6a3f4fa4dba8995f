"""Replay attention where its tiles begin and end: trajectory lengths around a step of 32 keys, a tile of 64, a query tile of
128 and a pass of 4096 positions of the list kernel; lists whose last step is partial, keys nobody sees, query tiles without
any key; a workspace full of garbage (list slots past a list's end hold whatever it held).

Against fp64 attention, 1e-4 absolute: the probabilities enter the second product with 2^-16 relative error against values
of at most ~5, the rest is fp32."""
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _check(B, T, Hq, Hkv, D, death, seed):
    import torch
    ngc = _ngc()
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(B, T, Hq, D), rnd(B, T, Hkv, D), rnd(B, T, Hkv, D)
    out = torch.full((B, T, Hq, D), float("nan"), device="cuda")
    ws = torch.full((ngc.ngc_replay_workspace_bytes(B, T, Hkv),), 0xFF, dtype=torch.uint8, device="cuda")
    scale = D ** -0.5
    print(f"[replay-edges] B={B} T={T} {Hq}/{Hkv} D={D} per_head={death.dim() == 3}", flush=True)
    ngc.ngc_replay_attn(q, k, v, death, B, T, Hq, Hkv, D, death.dim() == 3, scale, out, ws)
    torch.cuda.synchronize()
    i = torch.arange(T, device="cuda")
    for b in range(B):
        for h in range(Hkv):
            d = (death[b, h] if death.dim() == 3 else death[b]).long()
            vis = (i[None, :] <= i[:, None]) & (i[:, None] < d[None, :])
            kk, vv = k[b, :, h].double(), v[b, :, h].double()
            for x in range(Hq // Hkv):
                head = h * (Hq // Hkv) + x
                s = ((q[b, :, head].double() @ kk.t()) * scale).masked_fill(~vis, float("-inf"))
                p = torch.where(vis.any(1, keepdim=True), torch.softmax(s, -1), torch.zeros_like(s))
                assert (out[b, :, head].double() - p @ vv).abs().max() <= TOL, (b, h, head)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 161, 255, 257, 385])
def test_lengths_around_steps_and_tiles(T, D):
    import torch
    g = torch.Generator().manual_seed(T)
    death = torch.randint(1, 2 * T + 2, (2, 2, T), generator=g).to(torch.int32)     # any position, inside tiles too
    _check(2, T, 6, 2, D, death.cuda(), T)


@pytest.mark.parametrize("T", [4095, 4096, 4097, 8200])
def test_lengths_around_a_pass_of_the_list_kernel(T):
    import torch
    g = torch.Generator().manual_seed(T)
    round_of = (torch.arange(T) // 512 + 1) * 512
    death = torch.where(torch.rand(1, T, generator=g) < 0.7, round_of, torch.tensor(T)).to(torch.int32)
    _check(1, T, 2, 1, 128, death.cuda(), T)


def test_query_tiles_that_see_nothing_and_keys_nobody_sees():
    import torch
    T = 400
    death = torch.full((3, T), T, dtype=torch.int32)
    death[0] = 0                                   # nobody sees any key
    death[1, :] = torch.arange(T) + 1              # every query sees its own key only
    death[2, :300] = 256                           # the third query tile starts with an empty list ...
    death[2, 300:] = -5                            # ... and never gets a key
    _check(3, T, 3, 1, 128, death.cuda(), 1)
    _check(3, T, 4, 2, 64, death.cuda(), 2)
