"""Eq. 2 for given actions and its gradient at the edges of the route that holds a segment's row in LDS: row capacities
where the workgroup changes (1024, 2048, 8192, 16384 items), the pick bounds where it changes, the first length beyond the largest, rows that are
not 16-byte aligned, keep counts from one pick to all, masked entries, and segments that need the wide-range route in
between.  Against the fp64 oracle: log-probability 1e-4 relative, gradient 1e-4 of an entry plus 2e-6."""
import numpy as np
import pytest

import oracle as orc
from _harness import oracle_logprob

pytestmark = pytest.mark.gpu


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _segments(rng, stride, kmax):
    """(items, picks, kind) of the segments of one call."""
    full = min(stride, kmax)
    return [(stride, full, "normal"), (stride, 1, "normal"), (stride - 1, max(1, full // 3), "masked"),
            (max(1, stride // 2), min(full, max(1, stride // 2)), "normal"), (stride, max(1, full // 2), "wide"),
            (0, 0, "normal"), (min(stride, 5), min(full, 5), "normal"), (stride, max(1, full - 1), "normal")]


@pytest.mark.parametrize("stride", [7, 1023, 1024, 1025, 2048, 2051, 4096, 4097, 8192, 8193, 16384, 16385])
def test_rows_at_the_edges_of_their_capacities(stride):
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(stride)
    kmax = min(stride, 12000)
    segs = _segments(rng, stride, kmax)
    nseg = len(segs)
    n_items = np.array([s[0] for s in segs], np.int32)
    keep = np.array([s[1] for s in segs], np.int32)
    logits = np.full((nseg, stride), np.nan, np.float32)
    sigma = np.zeros((nseg, kmax), np.int32)
    gout = rng.standard_normal(nseg).astype(np.float32)
    for s, (n, k, kind) in enumerate(segs):
        if n == 0:
            continue
        x = rng.standard_normal(n).astype(np.float32)
        if kind == "wide":
            x[rng.random(n) < 0.2] -= np.float32(100.0)
        if kind == "masked" and n > 8:
            x[rng.choice(n, n // 8, replace=False)] = -np.inf
        logits[s, :n] = x
        order = rng.permutation(n)
        sigma[s, :k] = order[np.isfinite(x[order])][:k]
        keep[s] = min(k, int(np.isfinite(x).sum()))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    d_n, d_s, d_k, d_g = d(n_items), d(sigma), d(keep), d(gout)
    for shift in (0, 1):      # the second time every row starts 4 bytes later
        flat = torch.full((nseg * stride + 4,), float("nan"), device="cuda")
        x = flat[shift:shift + nseg * stride].view(nseg, stride)
        x.copy_(d(logits))
        out = torch.zeros(nseg, device="cuda")
        flat_g = torch.full((nseg * stride + 4,), float("nan"), device="cuda")
        grad = flat_g[shift:shift + nseg * stride].view(nseg, stride)
        print(f"[logprob-rows] stride={stride} shift={shift}", flush=True)
        ngc.ngc_subset_logprob(x, d_n, d_s, d_k, nseg, stride, kmax, out, ws)
        ngc.ngc_subset_logprob_backward(x, d_n, d_s, d_k, nseg, stride, kmax, kmax, d_g, grad, ws)
        torch.cuda.synchronize()
        lp, g = out.cpu().numpy(), grad.cpu().numpy()
        for s in range(nseg):
            n, k = int(n_items[s]), int(keep[s])
            if k == 0:
                assert lp[s] == 0.0
                continue
            assert lp[s] == pytest.approx(oracle_logprob(logits[s, :n], sigma[s, :k]), rel=1e-4, abs=1e-5), (s, n, k)
            assert np.isnan(g[s, n:]).all()
            if n * k <= 3_000_000:      # the oracle's gradient is term by term
                want = gout[s] * orc.logprob_grad(logits[s, :n], sigma[s, :k])
                assert np.all(np.abs(g[s, :n] - want) <= 1e-4 * np.abs(want) + 2e-6), (s, n, k)
            else:                       # what holds at any size: shift invariance, signs
                assert abs(g[s, :n].sum(dtype=np.float64)) <= 1e-3 * max(1.0, np.abs(g[s, :n]).sum(dtype=np.float64))
                picked = np.zeros(n, bool)
                picked[sigma[s, :k]] = True
                assert (g[s, :n][~picked] * gout[s] <= 0).all()
    assert all(v == 0 for v in ngc.read_status(ws))


def test_repeated_and_outlying_picks_are_counted_and_rows_may_be_shared():
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(3)
    n, k = 600, 40
    x = rng.standard_normal(n).astype(np.float32)
    sg = np.stack([rng.permutation(n)[:k] for _ in range(3)]).astype(np.int32)
    bad = sg.copy()
    bad[1, 7], bad[2, 3] = bad[1, 2], n + 5
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n_items, keep = d(np.full(3, n, np.int32)), d(np.full(3, k, np.int32))
    out = torch.zeros(3, device="cuda")
    ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    print("[logprob-rows] shared row", flush=True)
    ngc.ngc_subset_logprob(d(x), n_items, d(sg), keep, 3, 0, k, out, ws)      # stride 0: one row for all three
    assert all(v == 0 for v in ngc.read_status(ws))
    for s in range(3):
        assert float(out[s]) == pytest.approx(oracle_logprob(x, sg[s]), rel=1e-4)
    rows = d(np.stack([x] * 3))
    ngc.ngc_subset_logprob(rows, n_items, d(bad), keep, 3, n, k, out, ws)
    assert ngc.read_status(ws)[ngc.STATUS_BAD_SIGMA] == 2
    assert float(out[0]) == pytest.approx(oracle_logprob(x, sg[0]), rel=1e-4)
    assert bool(torch.isfinite(out).all())


@pytest.mark.parametrize("stride,kmax,nseg", [(16384, 1024, 513), (16384, 1025, 513), (16384, 2049, 513), (16384, 4097, 513),
                                              (16384, 4096, 512), (16384, 8193, 513), (8193, 1024, 513), (8192, 4097, 3),
                                              (16385, 4096, 3), (16388, 4097, 3), (16385, 8193, 3), (40000, 2048, 3),
                                              (0, 2048, 3), (0, 5000, 3)])
def test_workgroups_chosen_by_the_picks(stride, kmax, nseg):
    """Either side of every bound that decides about the workgroup beside the stride: picks and number of segments.  All
    segments but the last three are empty; of those, one fills the bound, one is short, one is as long as the stride (or, in
    longer strides, one item longer than what is held of a row in LDS)."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(stride + kmax)
    width = stride or 9000
    longest = width if stride and stride <= 16384 else 8065
    n_items, keep = np.zeros(nseg, np.int32), np.zeros(nseg, np.int32)
    n_items[-3:] = (min(width, kmax + 5), 37, longest) if stride else (8065, 8065, 8065)
    keep[-3:] = (min(kmax, n_items[-3]), 30, min(kmax, longest) - 1)
    logits = np.full((nseg if stride else 1, width), np.nan, np.float32)
    sigma = np.zeros((nseg, kmax), np.int32)
    row = lambda s: logits[s if stride else 0]
    for s in range(nseg - 3, nseg):
        if stride or s == nseg - 3:
            row(s)[:n_items[s]] = rng.standard_normal(n_items[s]).astype(np.float32)
        sigma[s, :keep[s]] = rng.permutation(n_items[s])[:keep[s]]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    x, d_n, d_s, d_k, out = d(logits), d(n_items), d(sigma), d(keep), torch.full((nseg,), float("nan"), device="cuda")
    gout = rng.standard_normal(nseg).astype(np.float32)
    ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    print(f"[logprob-rows] stride={stride} kmax={kmax} nseg={nseg}", flush=True)
    ngc.ngc_subset_logprob(x, d_n, d_s, d_k, nseg, stride, kmax, out, ws)
    lp = out.cpu().numpy()
    assert (lp[:-3] == 0).all()
    for s in range(nseg - 3, nseg):
        assert lp[s] == pytest.approx(oracle_logprob(row(s)[:n_items[s]], sigma[s, :keep[s]]), rel=1e-4, abs=1e-5), s
    if stride:
        grad = torch.full((nseg, stride), float("nan"), device="cuda")
        ngc.ngc_subset_logprob_backward(x, d_n, d_s, d_k, nseg, stride, kmax, kmax, d(gout), grad, ws)
        g = grad.cpu().numpy()
        assert np.isnan(g[:-3]).all()
        for s in range(nseg - 3, nseg):
            n, k = int(n_items[s]), int(keep[s])
            # the oracle's gradient is term by term; its cumulative form in fp64 serves where that takes too long
            if n * k <= 3_000_000:
                want = orc.logprob_grad(logits[s, :n], sigma[s, :k])
            else:
                e = np.exp(logits[s, :n].astype(np.float64) - logits[s, :n].max())
                picked = e[sigma[s, :k]]
                inv = np.cumsum(1.0 / (e.sum() - np.concatenate([[0.0], np.cumsum(picked)[:-1]])))
                want = -e * inv[-1]
                want[sigma[s, :k]] = 1.0 - picked * inv
            assert np.all(np.abs(g[s, :n] - gout[s] * want) <= 1e-4 * np.abs(gout[s] * want) + 2e-6 * max(1.0, abs(gout[s]))), (s, n, k)
            assert np.isnan(g[s, n:]).all()
    assert all(v == 0 for v in ngc.read_status(ws))


@pytest.mark.parametrize("stride,nseg", [(2049, 2049), (4096, 2049), (4096, 2048), (4097, 2049), (700, 5), (1500, 5), (4096, 5),
                                         (8192, 5), (8200, 600)])
def test_rows_held_in_registers(stride, nseg):
    """Rows as long as the threads hold and one item longer, either side of the number of segments that changes the
    workgroup: the last segments' rows end inside a group of four items, are picked to the last item, have masked and NaN
    entries (picked or not) or repeated and outlying picks; all other segments are empty."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(stride * 7 + nseg)
    kinds = ["all", "few", "masked", "masked pick", "repeated"]
    n_items, keep = np.zeros(nseg, np.int32), np.zeros(nseg, np.int32)
    logits = np.full((nseg, stride), np.nan, np.float32)
    sigma = np.full((nseg, stride), -7, np.int32)
    first = nseg - len(kinds)
    for i, kind in enumerate(kinds):
        s, n = first + i, stride - i
        x = rng.standard_normal(n).astype(np.float32)
        x[rng.integers(n)] -= 60.0
        if "masked" in kind:
            x[rng.choice(n, 9, replace=False)] = [-np.inf] * 5 + [np.nan] * 4
        order = rng.permutation(n)
        finite = order[np.isfinite(x[order])]
        k = {"all": n, "few": 3, "masked": n // 2}.get(kind, n // 3)
        sigma[s, :k] = (finite if "masked" in kind else order)[:k]
        if kind == "masked pick":
            sigma[s, k // 2] = order[~np.isfinite(x[order])][0]
        if kind == "repeated":
            sigma[s, 1], sigma[s, k - 1] = sigma[s, 0], stride + 3
        n_items[s], keep[s], logits[s, :n] = n, k, x
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    gout = rng.standard_normal(nseg).astype(np.float32)
    d_n, d_s, d_k, d_g = d(n_items), d(sigma), d(keep), d(gout)
    for shift in (0, 3):
        flat = torch.full((nseg * stride + 4,), float("nan"), device="cuda")
        x = flat[shift:shift + nseg * stride].view(nseg, stride)
        x.copy_(d(logits))
        out = torch.full((nseg,), float("nan"), device="cuda")
        grad = torch.full((nseg, stride), float("nan"), device="cuda")
        ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
        print(f"[logprob-rows] held stride={stride} nseg={nseg} shift={shift}", flush=True)
        ngc.ngc_subset_logprob(x, d_n, d_s, d_k, nseg, stride, stride, out, ws)
        assert ngc.read_status(ws)[ngc.STATUS_BAD_SIGMA] == 2
        ngc.ngc_subset_logprob_backward(x, d_n, d_s, d_k, nseg, stride, stride, stride, d_g, grad, ws)
        lp, g = out.cpu().numpy(), grad.cpu().numpy()
        assert (lp[:first] == 0).all() and np.isnan(g[:first]).all()
        for i, kind in enumerate(kinds):
            s = first + i
            n, k = int(n_items[s]), int(keep[s])
            assert np.isnan(g[s, n:]).all()
            if kind == "repeated":
                assert np.isfinite(lp[s]) and np.isfinite(g[s, :n]).all()
                continue
            if kind == "masked pick":
                assert lp[s] == -np.inf
                continue
            row = logits[s, :n].astype(np.float64)
            row[np.isnan(row)] = -np.inf
            e = np.exp(row - row.max())
            sig = sigma[s, :k]
            rest = np.cumsum(e[sig][::-1])[::-1] + np.delete(e, sig).sum()
            want = np.sum(row[sig] - row.max() - np.log(rest))
            # the total is rounded once; a term is off by 2^-21.6 and the ~40 roundings that R_j goes through one after the
            # other, 2.7e-6 at most.  Over many picks terms are ~log n - 1 >= 5 in the mean (5e-7 of them), three picks 8e-6
            assert abs(lp[s] - want) <= 1e-6 * abs(want) + 1e-5, (kind, n, k)
            c = np.cumsum(1.0 / rest)
            w = -e * c[-1]
            w[sig] = 1.0 - e[sig] * c
            assert np.all(np.abs(g[s, :n] - gout[s] * w) <= abs(gout[s]) * (1e-5 * np.abs(w) + 2e-6)), (kind, n, k)


@pytest.mark.parametrize("stride,n,nseg", [(16, 0, 192), (700, 700, 192), (4096, 3000, 192),     # held in registers
                                           (8200, 1500, 513),                                    # staged in LDS
                                           (16400, 8100, 96)])                                   # general route
def test_logprob_of_nearly_certain_given_picks(stride, n, nseg):
    """Ladders of picks, each far likelier than all that come after it, scattered over the row in a random order (n = 0: the
    row holds nothing else): log p is a small sum although logits lie up to 75 below the largest.  A pick's term is the
    logarithm of e_j / R_j, two fp32 numbers (2^-21.6 in all, 16 picks 5e-6), on every route.  1e-4 relative + 1e-5 as for
    any other row."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(stride)
    ladders = [(8, 10.0), (12, 6.5), (16, 5.0)]
    n_items, keep = np.zeros(nseg, np.int32), np.zeros(nseg, np.int32)
    logits, sigma = np.full((nseg, stride), np.nan, np.float32), np.zeros((nseg, 16), np.int32)
    want = np.zeros(nseg)
    for s in range(nseg):
        k, step = ladders[s % 3]
        m = n or k
        x = np.full(m, -79.9, np.float32)              # never picked
        sigma[s, :k] = rng.permutation(m)[:k]
        x[sigma[s, :k]] = -step * np.arange(k) + 0.01 * rng.random(k)
        x += np.float32(3.0)
        n_items[s], keep[s], logits[s, :m] = m, k, x
        e = np.exp(x.astype(np.float64) - x.max())
        rest = np.cumsum(e[sigma[s, :k]][::-1])[::-1] + np.delete(e, sigma[s, :k]).sum()
        want[s] = np.sum(np.log(e[sigma[s, :k]] / rest))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.zeros(nseg, device="cuda")
    ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    print(f"[logprob-rows] ladder stride={stride} n={n} nseg={nseg}", flush=True)
    ngc.ngc_subset_logprob(d(logits), d(n_items), d(sigma), d(keep), nseg, stride, 16, out, ws)
    off = np.abs(out.cpu().numpy() - want)
    assert np.all(off <= 1e-4 * np.abs(want) + 1e-5), (off.max(), int((off > 1e-4 * np.abs(want) + 1e-5).sum()))


@pytest.mark.parametrize("stride,n,nseg", [(64, 64, 4), (8200, 1500, 513)])        # held in registers, staged in LDS
def test_gradient_with_large_upstream_weights(stride, n, nseg):
    """Upstream weights as a loss scale makes them, over rows whose last items lie just under 80 below the largest: the sum of
    1 / R_j reaches e^80, its product with the weight leaves fp32's range, the gradient (weight times a share) does not.
    Masked items that nobody picks get 0.  1e-4 of an entry plus 2e-6 of the weight as elsewhere."""
    import torch
    ngc = _ngc()
    rng = np.random.default_rng(n)
    first, k = nseg - 3, n // 2
    weights = np.array([65536.0, -1.0e6, 1.0e-3], np.float32)
    n_items, keep, gout = np.zeros(nseg, np.int32), np.zeros(nseg, np.int32), np.zeros(nseg, np.float32)
    logits, sigma = np.full((nseg, stride), np.nan, np.float32), np.zeros((nseg, k), np.int32)
    for s in range(first, nseg):
        order = rng.permutation(n)
        x = np.full(n, -79.5, np.float32) + 0.1 * rng.random(n).astype(np.float32)
        x[order[0]] = 0.0
        x[order[-3:]] = -np.inf
        n_items[s], keep[s], gout[s], logits[s, :n], sigma[s] = n, k, weights[s - first], x, order[:k]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    grad = torch.full((nseg, stride), float("nan"), device="cuda")
    ws = torch.zeros(ngc.STATUS_WORDS * 4, dtype=torch.uint8, device="cuda")
    print(f"[logprob-rows] large weights stride={stride} n={n}", flush=True)
    ngc.ngc_subset_logprob_backward(d(logits), d(n_items), d(sigma), d(keep), nseg, stride, k, k, d(gout), grad, ws)
    g = grad.cpu().numpy()
    for s in range(first, nseg):
        e = np.exp(logits[s, :n].astype(np.float64))
        picked = e[sigma[s]]
        inv = np.cumsum(1.0 / (np.cumsum(picked[::-1])[::-1] + np.delete(e, sigma[s]).sum()))
        want = -e * inv[-1]
        want[sigma[s]] = 1.0 - picked * inv
        assert np.all(np.abs(g[s, :n] - gout[s] * want) <= abs(gout[s]) * (1e-4 * np.abs(want) + 2e-6)), s
        assert (g[s, :n][np.isinf(logits[s, :n])] == 0).all() and np.isnan(g[s, n:]).all()
