"""A pooled round's routes: ranking in LDS and selection by radix, rows moved by the selecting workgroup and by a second
launch, both workgroup sizes, at the sizes where they change and on keys that send a sequence from ranking to radix.  Kept
lists, sampled orders, lengths, rows and positions are the oracle's, bit for bit; log-probabilities 1e-4 relative (fp32 sums
of up to 16384 terms, measured 1e-6)."""
import numpy as np
import pytest

import oracle as orc
from _harness import oracle_logprob

pytestmark = pytest.mark.gpu


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _logits(rng, n, kind):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "equal":
        x[:] = np.float32(0.25)
    elif kind == "masked" and n:
        x[rng.random(n) < 0.67] = -np.inf
    elif kind == "nan" and n:
        x[rng.integers(n)] = np.nan
    elif kind == "wide" and n:
        x *= np.float32(60)
    return x


def _round(L, B, H, cap, D, lens, keeps, max_keep, kinds, tau=1.0, layer=-1, select_only=False, outputs=True):
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(1000 * B + 10 * H + cap)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    logits = np.zeros((L, B, H, cap), np.float32)
    for l in range(L):
        for b in range(B):
            for h in range(H):
                logits[l, b, h, :lens[l, b, h]] = _logits(rng, int(lens[l, b, h]), kinds[b % len(kinds)])
    c = ngc.Cache.allocate(L, B, H, H, D, cap, with_pos=True)
    rows = torch.randint(-200, 200, (L, B, H, cap, D), device="cuda", dtype=torch.int32,
                         generator=torch.Generator("cuda").manual_seed(cap)).to(torch.bfloat16)
    c.k.copy_(rows)
    c.v.copy_(-rows)
    c.pos.copy_(torch.arange(cap, device="cuda", dtype=torch.int32).expand(L, B, H, cap) * 3)
    c.len.copy_(d(lens))
    ws = torch.zeros(ngc.ngc_workspace_bytes(c, max_keep) + 16 * L * B * H * cap, dtype=torch.uint8, device="cuda")
    kept = torch.full((L, B, H, max_keep), -1, dtype=torch.int32, device="cuda")
    sigma = torch.full_like(kept, -1) if outputs else None
    logp = torch.full((L, B, H), 7.0, device="cuda") if outputs else None
    p = ngc.make_params(noise_scale=tau, round=4, seed=77,
                        flags=ngc.EVICT_POOL_HEADS | (ngc.EVICT_SELECT_ONLY if select_only else 0))
    print(f"[pooled-routes] L={L} B={B} H={H} cap={cap} D={D} tau={tau} layer={layer} select_only={select_only}", flush=True)
    ngc.ngc_evict(c, layer, d(logits), d(keeps), p, max_keep, kept, sigma, logp, ws)
    torch.cuda.synchronize()
    assert all(x == 0 for x in ngc.read_status(ws))
    hk, hn = kept.cpu().numpy(), c.len.cpu().numpy()
    hs, hl = (sigma.cpu().numpy(), logp.cpu().numpy()) if outputs else (None, None)
    k0, k1, v1, p1 = rows.cpu().float().numpy(), c.k.cpu().float().numpy(), c.v.cpu().float().numpy(), c.pos.cpu().numpy()
    for l in range(L):
        for b in range(B):
            if layer not in (-1, l):
                assert (hn[l, b] == lens[l, b]).all() and (hk[l, b] == -1).all()
                assert (k1[l, b] == k0[l, b]).all()
                continue
            heads = [logits[l, b, h, :lens[l, b, h]] for h in range(H)]
            heads = [np.where(np.isnan(x), np.float32(-np.inf), x) for x in heads]      # a NaN counts as masked
            K = int(keeps[l, b].sum())
            want, osig, cat, osig_idx = orc.evict_select_pooled(heads, K, tau, 77, 4, l, b)
            for h in range(H):
                n = len(want[h])
                assert hk[l, b, h, :n].tolist() == want[h].tolist(), (l, b, h)
                assert (hk[l, b, h, n:] == -1).all()
                if select_only:
                    assert hn[l, b, h] == lens[l, b, h] and (k1[l, b, h] == k0[l, b, h]).all()
                    continue
                assert hn[l, b, h] == n
                assert (k1[l, b, h, :n] == k0[l, b, h, want[h]]).all() and (v1[l, b, h, :n] == -k0[l, b, h, want[h]]).all()
                assert p1[l, b, h, :n].tolist() == (3 * want[h]).tolist()
            if not outputs:
                continue
            assert hs[l, b].reshape(-1)[:K].tolist() == [h * cap + t for h, t in osig], (l, b)
            lp = oracle_logprob(cat, osig_idx) if K else 0.0
            assert (hl[l, b, 1:] == 0).all()
            if np.isfinite(lp):
                assert hl[l, b, 0] == pytest.approx(lp, rel=1e-4, abs=1e-5), (l, b)
            else:
                assert hl[l, b, 0] == lp, (l, b)


def _ragged(rng, L, B, H, cap, share=0.5):
    lens = rng.integers(max(1, cap // 2), cap + 1, (L, B, H)).astype(np.int32)
    if H > 1:
        lens[:, 0, H - 1] = 0                          # an empty head among others
    lens[:, -1] = cap
    return lens, np.ceil(lens * share).astype(np.int32)


# one and two launches (128 sequences), 512 threads (beyond 256, up to 2560 items), head counts, row counts off four
@pytest.mark.parametrize("L,B,H,cap,D", [(1, 1, 1, 5, 64), (1, 2, 16, 9, 64), (2, 3, 2, 257, 128), (1, 128, 2, 41, 64),
                                         (1, 129, 2, 41, 64), (1, 256, 2, 30, 64), (1, 257, 3, 30, 128),
                                         (1, 257, 8, 320, 64), (1, 257, 8, 321, 64), (1, 3, 5, 1023, 128)])
def test_launches_and_workgroups(L, B, H, cap, D):
    lens, keeps = _ragged(np.random.default_rng(cap + B), L, B, H, cap)
    _round(L, B, H, cap, D, lens, keeps, cap, ["normal"])


# two heads: 160 KB hold 33536 bytes of 1024 threads, 6 and a bit for every item that is ranked and 2 for each that may be kept.
# With all of them kept 16032 items (163800 of 163840 bytes), with 2 x 3000 19200 (163136); the next sizes go by radix.
@pytest.mark.parametrize("cap,max_keep,share,kinds", [
    (8016, 8016, 1.0, ["normal"]), (8020, 8020, 1.0, ["normal"]), (9600, 3000, 0.25, ["normal"]), (9700, 3000, 0.25, ["normal"]),
    (8013, 8013, 0.5, ["equal", "masked"]), (8192, 8192, 1.0, ["normal"]), (8191, 3000, 0.25, ["normal"]),
    (8700, 3000, 0.25, ["normal"]), (9001, 9001, 0.5, ["normal"])])
def test_items_in_lds_and_beyond(cap, max_keep, share, kinds):
    lens, keeps = _ragged(np.random.default_rng(cap), 1, 2, 2, cap, share)
    _round(1, 2, 2, cap, 64, lens, keeps, max_keep, kinds)


@pytest.mark.parametrize("tau", [0.0, 1.0])
@pytest.mark.parametrize("B", [5, 260])
def test_keys_that_are_not_ranked(B, tau):
    """Many equal keys, masked entries kept, NaN, a wide spread: next to sequences that are ranked."""
    rng = np.random.default_rng(B)
    lens, keeps = _ragged(rng, 1, B, 2, 203)
    keeps[0, 3] = lens[0, 3]                           # everything, the masked entries too
    keeps[0, 4] = 0
    _round(1, B, 2, 203, 64, lens, keeps, 203, ["normal", "equal", "nan", "masked", "wide"], tau)


@pytest.mark.parametrize("B", [4, 140])
def test_one_layer_selection_alone_and_no_outputs(B):
    lens, keeps = _ragged(np.random.default_rng(B), 2, B, 2, 66)
    _round(2, B, 2, 66, 64, lens, keeps, 66, ["normal"], layer=1)
    _round(2, B, 2, 66, 64, lens, keeps, 66, ["normal"], select_only=True)
    _round(2, B, 2, 66, 64, lens, keeps, 66, ["normal"], outputs=False)
