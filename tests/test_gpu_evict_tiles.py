"""Rounds that move rows, at the sizes where the copy changes: a tile of rows and one more or less, blocks that are powers of
two and blocks that are not, either side of the rows, segments and kept share that choose the workgroup, logits beyond what a
thread keeps in registers.  Kept list, sampled order and log-probability against the same round in selection-only mode (which
other tests compare with the oracle), rows against a gather of the original ones by the kept list."""
import pytest

pytestmark = pytest.mark.gpu


def _ngc():
    from paper_2604_18002_amd import binding
    binding.load_library()
    return binding


def _round(ngc, L, B, Hkv, cap, D, block, n, keep, max_keep, logits, flags, k, v, pos):
    import torch
    cache = ngc.Cache(k.clone(), v.clone(), n.clone(), pos.clone(), 2 * Hkv)
    kept = torch.full((L, B, Hkv, max_keep), -7, dtype=torch.int32, device="cuda")
    sigma, logp = torch.full_like(kept, -7), torch.zeros(L, B, Hkv, device="cuda")
    ws = ngc.allocate_workspace(cache, max_keep)
    p = ngc.make_params(block=block, noise_scale=1.0, round=3, seed=11, flags=flags)
    ngc.ngc_evict(cache, -1, logits, keep, p, max_keep, kept, sigma, logp, ws)
    assert all(x == 0 for x in ngc.read_status(ws))
    return cache, kept, sigma, logp


@pytest.mark.parametrize("nseg,cap,block,D,num,den", [
    # 256 threads: tiles of 96 rows (192 of 128 bytes)
    (4, 200, 1, 128, 95, 200), (4, 200, 1, 128, 97, 200), (4, 400, 1, 64, 1, 2), (6, 512, 3, 128, 1, 2),
    # 512 threads: tiles of 256 rows (512)
    (4, 513, 1, 128, 255, 513), (4, 600, 1, 128, 257, 600), (4, 1100, 2, 128, 512, 1100), (4, 1537, 5, 64, 1, 3),
    (4, 2200, 32, 128, 1, 2), (3, 4096, 1, 128, 9, 10),
    # 1024 threads beyond 4096 rows, and below with many segments or most rows kept
    (3, 4097, 1, 128, 256, 4097), (3, 4500, 7, 64, 1, 2), (3, 9000, 1, 128, 2, 5), (514, 1537, 1, 64, 1, 2),
    (514, 1536, 1, 64, 1, 2), (1026, 1281, 1, 64, 1, 2), (1026, 1281, 1, 64, 1, 3), (1538, 1281, 1, 64, 1, 3),
    (1538, 1280, 1, 64, 1, 3),
    # either side of the kept share that decides: half of the rows, a third beyond 2048 segments
    (514, 1537, 1, 64, 769, 1537), (514, 1537, 1, 64, 768, 1537), (1026, 1281, 1, 64, 641, 1281),
    (1026, 1281, 1, 64, 640, 1281), (2050, 1281, 1, 64, 427, 1281), (2050, 1281, 1, 64, 426, 1281),
    (2048, 1281, 1, 64, 427, 1281), (2050, 1290, 3, 128, 143, 430), (514, 1540, 4, 128, 193, 385)])
def test_rows_follow_the_kept_list(nseg, cap, block, D, num, den):
    import torch
    ngc = _ngc()
    L, Hkv = 1, 2
    B = nseg // 2 if nseg % 2 == 0 else nseg
    if nseg % 2:
        Hkv = 1
    g = torch.Generator(device="cuda").manual_seed(nseg * 7 + cap)
    rnd = lambda *s: torch.randint(-2 ** 15, 2 ** 15, s, generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16)
    k, v = rnd(L, B, Hkv, cap, D), rnd(L, B, Hkv, cap, D)
    pos = torch.arange(cap, device="cuda", dtype=torch.int32).expand(L, B, Hkv, cap).contiguous()
    n = torch.full((L, B, Hkv), cap, dtype=torch.int32, device="cuda")
    n[0, B // 2:, -1] -= cap // 3 + 1                       # some end inside a block
    items_cap = -(-cap // block)
    max_keep = -(-items_cap * num // den)                   # the bound that the workgroup is chosen by
    n[0, -1, -1] = block * max_keep // 2 + 1
    items = (n + block - 1) // block
    keep = torch.minimum((items * num + den - 1) // den, items).clamp(min=1).to(torch.int32)
    keep[0, 0, 0] = 1
    keep[0, -1, -1] = items[0, -1, -1]                      # nothing moves
    assert int(keep.max()) <= max_keep
    logits = torch.randn(L, B, Hkv, cap, generator=g, device="cuda")
    print(f"[evict-tiles] nseg={nseg} cap={cap} block={block} D={D} {num}/{den}", flush=True)
    args = (L, B, Hkv, cap, D, block, n, keep, max_keep, logits)
    cache, kept, sigma, logp = _round(ngc, *args, 0, k, v, pos)
    _, kept_s, sigma_s, logp_s = _round(ngc, *args, ngc.EVICT_SELECT_ONLY, k, v, pos)
    assert torch.equal(kept, kept_s) and torch.equal(sigma, sigma_s)
    # both add up the same terms, in chunks that depend on the workgroup
    assert torch.all((logp - logp_s).abs() <= 1e-6 * logp_s.abs() + 1e-4)
    rows = torch.arange(max_keep * block, device="cuda")
    item = kept.clamp(min=0).long().gather(-1, (rows // block).expand(L, B, Hkv, -1))
    src = item * block + rows % block                       # source row of every row after the round
    last = kept.long().gather(-1, keep.long().unsqueeze(-1) - 1).squeeze(-1)
    short = torch.where(last == items - 1, items * block - n, torch.zeros_like(n))
    want_len = keep * block - short
    assert torch.equal(cache.len, want_len.to(torch.int32))
    live = rows < want_len.unsqueeze(-1)
    src = torch.where(live, src, torch.zeros_like(src))
    width = min(cap, max_keep * block)
    src, live = src[..., :width], live[..., :width]
    for got, orig in ((cache.k, k), (cache.v, v)):
        moved = orig.view(torch.int16).gather(3, src.unsqueeze(-1).expand(*src.shape, D))
        same = (got.view(torch.int16)[..., :width, :] == moved).all(-1)
        assert bool((same | ~live).all())
    assert bool(((cache.pos[..., :width] == src) | ~live).all())
