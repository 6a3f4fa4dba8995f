"""The selection's routes (ranking by buckets, radix select, ranking by all pairs) at the item counts where they change and
on keys that send a segment from one to another: many equal keys, masked entries, infinities, ranges that overflow, every
keep count from one to all, with and without noise, at the three workgroup sizes.  Kept lists and sampled orders are the
oracle's, bit for bit; log-probabilities 1e-4 relative."""
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
    if kind == "equal":            # one bucket holds more than any ranking by buckets takes
        x[:] = np.float32(0.25)
    elif kind == "quantised":
        x = (np.round(x * 2) / 2).astype(np.float32)
    elif kind == "masked":         # two thirds masked
        x[rng.random(n) < 0.67] = -np.inf
    elif kind == "few-masked":
        x[rng.choice(n, min(n - 1, 20), replace=False)] = -np.inf
    elif kind == "all-masked":
        x[:] = -np.inf
    elif kind == "infinite":
        x[rng.integers(n)] = np.inf
    elif kind == "huge":           # the value range of the keys is infinite in fp32
        x[rng.integers(n)] = np.float32(3e38)
        x[rng.integers(n)] = np.float32(-3e38)
    elif kind == "outlier":        # nearly everything in one bucket
        x[rng.integers(n)] = np.float32(1e6)
    elif kind == "signed-zero":
        x = np.where(rng.random(n) < 0.5, np.float32(-0.0), np.float32(0.0)).astype(np.float32)
        x[: n // 2] += rng.standard_normal(n // 2).astype(np.float32)
    return x


KINDS = ["normal", "equal", "quantised", "masked", "few-masked", "all-masked", "infinite", "huge", "outlier", "signed-zero"]


@pytest.mark.parametrize("tau", [0.0, 1.0])
@pytest.mark.parametrize("cap", [64, 65, 96, 127, 128, 129, 255, 256, 257, 513, 700, 2048, 2049, 4099, 8200])
def test_routes_agree_with_the_oracle(cap, tau):
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(cap)
    B, D, seed, rnd = len(KINDS), 64, 99, 3
    lens = np.array([cap - (i % 3) for i in range(B)], np.int32)
    keeps = np.array([max(1, n // 2) for n in lens], np.int32)
    keeps[0], keeps[2], keeps[4], keeps[9] = lens[0], 1, lens[4] - 1, lens[9]
    logits = np.zeros((1, B, 1, cap), np.float32)
    for b, kind in enumerate(KINDS):
        logits[0, b, 0, :lens[b]] = _logits(rng, lens[b], kind)
    mk = int(keeps.max())
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for flags in (ngc.EVICT_SELECT_ONLY, 0, ngc.EVICT_UNORDERED):
        c = ngc.Cache.allocate(1, B, 1, 1, D, cap)
        rows = torch.arange(cap, device="cuda").remainder(251).to(torch.bfloat16)
        c.k.copy_(rows.view(1, 1, 1, cap, 1).expand_as(c.k))
        c.v.copy_(c.k)
        c.len.copy_(d(lens.reshape(1, B, 1)))
        ws = ngc.allocate_workspace(c, mk)
        kept = torch.full((1, B, 1, mk), -1, dtype=torch.int32, device="cuda")
        sigma, logp = torch.full_like(kept, -1), torch.full((1, B, 1), float("nan"), device="cuda")
        p = ngc.make_params(noise_scale=tau, round=rnd, seed=seed, flags=flags)
        print(f"[select-routes] cap={cap} tau={tau} flags={flags}", flush=True)
        ngc.ngc_evict(c, -1, d(logits), d(keeps.reshape(1, B, 1)), p, mk, kept, sigma, logp, ws)
        torch.cuda.synchronize()
        hk, hs, hl = kept.cpu().numpy()[0, :, 0], sigma.cpu().numpy()[0, :, 0], logp.cpu().numpy()[0, :, 0]
        for b, kind in enumerate(KINDS):
            n, K = int(lens[b]), int(keeps[b])
            x = logits[0, b, 0, :n]
            want_k, want_s = orc.evict_select(x, K, tau, seed, rnd, 0, b, 0)
            assert (hk[b, :K] == want_k).all(), (kind, n, K)
            assert (hs[b, :K] == want_s).all(), (kind, n, K)
            assert (hk[b, K:] == -1).all() and (hs[b, K:] == -1).all()
            if kind == "infinite":
                continue                              # Eq. 2 is not defined there
            # (the short form of the oracle leaves the range of fp64 beyond spans of ~745)
            want = orc.logprob_literal(x, want_s) if kind in ("huge", "outlier") else oracle_logprob(x, want_s)
            if np.isinf(want):
                assert hl[b] == want, (kind, n, K)
            else:
                assert hl[b] == pytest.approx(want, rel=1e-4, abs=1e-5), (kind, n, K)
            if flags == 0:
                assert torch.equal(c.k[0, b, 0, :K, 0], rows[torch.from_numpy(want_k).long().cuda()])
        assert all(v == 0 for v in ngc.read_status(ws))


@pytest.mark.parametrize("tail", ["spread", "equal"])      # ranking by buckets; too many equal keys: the other routes
@pytest.mark.parametrize("n", [0, 70, 256, 700, 2100, 9000])
def test_logprob_of_nearly_certain_picks(n, tail):
    """A ladder of picks, each far likelier than all that come after it: log p is a small sum of differences of large
    numbers (logits up to 80 below the largest).  A pick's term in a round's log-probability is log(e_j / R_j) of two fp32
    numbers: e_j and R_j are rounded (2 x 2^-24), so are the two mantissa products and their quotient (3 x 2^-24): 2^-21.6
    in all.  So is a pick's term of Eq. 2 for given picks.  Beyond that the 1e-4 relative that holds everywhere."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(n)
    ladders = [(17, 4.9), (12, 6.6), (30, 2.7), (9, 9.7)]
    cap = max(n, 30)
    lens = np.array([n or k for k, _ in ladders], np.int32)
    keeps = np.array([k for k, _ in ladders], np.int32)
    if n:
        keeps[:2] -= 2                                     # what lies lowest is the tail, never picked
    B, mk = len(ladders), int(keeps.max())
    logits = np.zeros((1, B, 1, cap), np.float32)
    for b, (k, step) in enumerate(ladders):
        x = np.full(lens[b], -79.9, np.float32)            # a span of just under 80: no wide-range route
        if tail == "spread":
            x += rng.random(lens[b]).astype(np.float32)
        x[rng.permutation(lens[b])[:k]] = -step * np.arange(k) + 0.01 * rng.random(k)
        logits[0, b, 0, :lens[b]] = x - x.max() + np.float32(3.0)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d_x, d_keep, d_len = d(logits), d(keeps.reshape(1, B, 1)), d(lens.reshape(1, B, 1))
    for flags in (ngc.EVICT_SELECT_ONLY, 0):
        c = ngc.Cache.allocate(1, B, 1, 1, 64, cap)
        c.len.copy_(d_len)
        ws = ngc.allocate_workspace(c, mk)
        kept = torch.zeros((1, B, 1, mk), dtype=torch.int32, device="cuda")
        sigma, logp = torch.zeros_like(kept), torch.zeros((1, B, 1), device="cuda")
        given = torch.zeros(B, device="cuda")
        print(f"[select-routes] ladder n={n} tail={tail} flags={flags}", flush=True)
        ngc.ngc_evict(c, -1, d_x, d_keep, ngc.make_params(noise_scale=0.0, flags=flags), mk, kept, sigma, logp, ws)
        ngc.ngc_subset_logprob(d_x, d_len, sigma, d_keep, B, cap, mk, given, ws)
        torch.cuda.synchronize()
        hs = sigma.cpu().numpy()[0, :, 0]
        for b in range(B):
            x, K = logits[0, b, 0, :lens[b]], int(keeps[b])
            _, want_s = orc.evict_select(x, K, 0.0, 0, 0, 0, b, 0)
            assert (hs[b, :K] == want_s).all()
            want = oracle_logprob(x, want_s)
            for got in (float(logp[0, b, 0]), float(given[b])):
                assert abs(got - want) <= 1e-4 * abs(want) + K * 2.0 ** -21.6, (n, tail, b, got, want)
        assert all(v == 0 for v in ngc.read_status(ws))


@pytest.mark.parametrize("cap,max_keep,fits", [(16384, 15225, True), (16384, 15232, True), (16384, 15233, True),
                                               (16104, 16088, True), (16352, 16352, True), (16384, 16320, True),
                                               (16384, 16321, False)])
def test_selections_that_fill_the_lds(cap, max_keep, fits):
    """Up to the documented limit, and just beyond it; with buckets and index buffers the first four ask for 160 KB or a
    few bytes less."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(max_keep)
    x = rng.standard_normal((1, 1, 2, cap)).astype(np.float32)
    keeps = np.array([max_keep, cap // 3], np.int32)
    for flags in (ngc.EVICT_SELECT_ONLY, 0):
        c = ngc.Cache.allocate(1, 1, 2, 2, 64, cap)
        c.len.fill_(cap)
        ws = ngc.allocate_workspace(c, max_keep)
        kept = torch.zeros((1, 1, 2, max_keep), dtype=torch.int32, device="cuda")
        sigma, logp = torch.zeros_like(kept), torch.zeros((1, 1, 2), device="cuda")
        args = (c, -1, torch.from_numpy(x).cuda(), torch.from_numpy(keeps.reshape(1, 1, 2)).cuda(),
                ngc.make_params(seed=5, flags=flags), max_keep, kept, sigma, logp, ws)
        print(f"[select-routes] lds cap={cap} max_keep={max_keep} flags={flags}", flush=True)
        if not fits:
            with pytest.raises(ngc.NgcError) as e:
                ngc.ngc_evict(*args)
            assert e.value.code == ngc.NGC_EUNSUPPORTED
            continue
        ngc.ngc_evict(*args)
        torch.cuda.synchronize()
        for h in range(2):
            want_k, want_s = orc.evict_select(x[0, 0, h], int(keeps[h]), 1.0, 5, 0, 0, 0, h)
            assert (kept[0, 0, h, :keeps[h]].cpu().numpy() == want_k).all()
            assert (sigma[0, 0, h, :keeps[h]].cpu().numpy() == want_s).all()
            assert float(logp[0, 0, h]) == pytest.approx(oracle_logprob(x[0, 0, h], want_s), rel=1e-4)
        assert c.len.flatten().tolist() == ([cap, cap] if flags else keeps.tolist())
        assert all(v == 0 for v in ngc.read_status(ws))


@pytest.mark.parametrize("tau", [0.0, 1.0])
@pytest.mark.parametrize("cap", [65, 200, 700, 2100, 8200])
def test_masked_items_rank_behind_all_others(cap, tau):
    """Many masked items (-inf and NaN), keep counts below, at and above the number of unmasked ones: the ranking by buckets
    takes the first two, the others the rest; a single unmasked item, and none."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(cap)
    shares = [0.3, 0.5, 0.5, 0.5, 0.9, 0.98, None, 1.0]         # masked share; None: one unmasked item
    extra = [-1, -1, 0, 1, -1, 0, 0, 3]                         # keep count minus the unmasked ones
    B = len(shares)
    logits, lens = np.zeros((1, B, 1, cap), np.float32), np.full(B, cap, np.int32)
    keeps = np.zeros(B, np.int32)
    for b, share in enumerate(shares):
        x = rng.standard_normal(cap).astype(np.float32)
        x[rng.random(cap) < (1.0 if share is None else share)] = -np.inf
        if share is None:
            x[cap // 2] = 1.0
        unmasked = int(np.isfinite(x).sum())
        x[np.isinf(x) & (rng.random(cap) < 0.2)] = np.nan
        logits[0, b, 0], keeps[b] = x, max(1, unmasked + extra[b])
    mk = int(keeps.max())
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    c = ngc.Cache.allocate(1, B, 1, 1, 64, cap)
    c.len.copy_(d(lens.reshape(1, B, 1)))
    ws = ngc.allocate_workspace(c, mk)
    kept = torch.full((1, B, 1, mk), -1, dtype=torch.int32, device="cuda")
    sigma, logp = torch.full_like(kept, -1), torch.full((1, B, 1), float("nan"), device="cuda")
    print(f"[select-routes] masked cap={cap} tau={tau}", flush=True)
    ngc.ngc_evict(c, -1, d(logits), d(keeps.reshape(1, B, 1)), ngc.make_params(noise_scale=tau, seed=7, round=1), mk, kept,
                  sigma, logp, ws)
    torch.cuda.synchronize()
    for b in range(B):
        x, K = np.where(np.isnan(logits[0, b, 0]), np.float32(-np.inf), logits[0, b, 0]), int(keeps[b])
        want_k, want_s = orc.evict_select(x, K, tau, 7, 1, 0, b, 0)
        assert (kept[0, b, 0, :K].cpu().numpy() == want_k).all(), (b, K)
        assert (sigma[0, b, 0, :K].cpu().numpy() == want_s).all(), (b, K)
        got = float(logp[0, b, 0])
        if np.isneginf(x[want_s]).any():
            assert got == -np.inf, (b, K)
        else:
            assert got == pytest.approx(oracle_logprob(x, want_s), rel=1e-4, abs=1e-5), (b, K)
    assert all(v == 0 for v in ngc.read_status(ws))
