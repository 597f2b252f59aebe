"""The launches of the multi-launch plans at the edges of their shapes.

Attention (``retro_decode_attend``) against a plain fp64 softmax over the selected
tokens, in the streamed kernel (64 KV heads a sequence) and in the one that stages
chunks through LDS (2): every number of row tiles a wavefront arrangement takes,
both page sizes and head dimensions, odd page counts (a chunk with one page), a half-filled last
page, pages that past rows may not use, unmapped pages, and cache slots past the
sequence filled with NaN.  Selection: the rows of ``retro_select_pages`` and of a
step's attention launch against a stable sort of the scores they report, at
table lengths on both sides of every stripe count.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _layer(**kw):
    from paper_2508_09001_amd.layer import RetroLayer
    base = dict(batch=2, num_kv_heads=2, group=4, head_dim=128, page_size=16, budget=512,
                window=3, max_pages=70)
    base.update(kw)
    return RetroLayer(**base)


# (W + 1) * G rows: 1, 2, 3, 4, 5, 6, 7 (two groups of tiles) and 17 tiles of 16
TILES = {(0, 1): 1, (3, 5): 2, (16, 2): 3, (15, 4): 4, (16, 4): 5, (10, 8): 6, (16, 6): 4,
         (64, 4): 6}


@pytest.mark.parametrize("hk", [2, 64])
@pytest.mark.parametrize("W,G", sorted(TILES))
@pytest.mark.parametrize("P,d", [(16, 128), (32, 128), (16, 64), (32, 64)])
def test_attend_matches_fp64(W, G, P, d, hk):
    from paper_2508_09001_amd import binding as B
    pages, mp, t = 33, 40, 200
    lay = _layer(num_kv_heads=hk, group=G, window=W, head_dim=d, page_size=P, budget=pages * P,
                 max_pages=mp, num_phys_pages=2 * mp)
    # splits of nine chunks or more with 64 heads: always the streamed kernel's
    tiles = B.retro_attend_plan(lay.dims, False)[0]
    assert tiles in ((0, TILES[W, G]) if hk == 2 else (TILES[W, G],))
    g = torch.Generator().manual_seed(W * 100 + G + P + d + hk - 2)
    b, hq = 2, hk * G

    def rand(*s):
        return torch.randn(*s, generator=g)

    lens = torch.tensor([mp * P - P // 2 - 3, 20 * P + 1])
    keys, vals = rand(b, mp, hk, P, d), rand(b, mp, hk, P, d)
    pos = torch.arange(mp * P).view(mp, P)
    for s in range(b):                       # slots that hold no token
        keys[s][(pos >= lens[s])[:, None].expand(mp, hk, P)] = float("nan")
        vals[s][(pos >= lens[s])[:, None].expand(mp, hk, P)] = float("nan")
    keys, vals = keys.bfloat16(), vals.bfloat16()
    lay.k_cache.copy_(keys.view(b * mp, hk, P, d))
    lay.v_cache.copy_(vals.view(b * mp, hk, P, d).transpose(2, 3))
    lay.page_table[0, 7] = -1                # a selected page that is not mapped: skipped
    lay.seq_lens.copy_(lens)
    nsel = torch.tensor([[pages, 4], [21, 1]]).repeat(1, hk // 2)
    sel = torch.full((b, hk, pages), -1, dtype=torch.int32)
    msk = torch.full((b, hk, pages), -1, dtype=torch.int32)
    for s in range(b):
        n_pages = -(-int(lens[s]) // P)
        for h in range(hk):
            k = int(nsel[s, h])
            # the first page and the half-filled last one are always among them
            rest = torch.randperm(n_pages - 2, generator=g)[:max(k - 2, 0)] + 1
            p = torch.cat([torch.tensor([n_pages - 1]), rest, torch.tensor([0])])[:k].sort().values
            sel[s, h, :k] = p.int()
            ago = torch.randint(1, W + 5, (k,), generator=g)
            msk[s, h, :k] = torch.where(torch.rand(k, generator=g) < 0.5, t - ago, -1).int()
    lay.selected.copy_(sel)
    lay.mask.copy_(msk)
    lay.num_selected.copy_(nsel)
    q = rand(b, W + 1, hq, d).bfloat16()
    print(f"[stream] hk={hk} W={W} G={G} P={P} d={d}", flush=True)
    lay.attend(t, q.cuda())
    torch.cuda.synchronize()
    o, z = lay.o_part.cpu().double(), lay.lse_part.cpu().double()
    taus = torch.arange(W + 1) + t - W
    for s in range(b):
        for h in sorted({0, 1, hk - 2, hk - 1}):
            k = int(nsel[s, h])
            p = sel[s, h, :k].long()
            ok = ((pos[p] < lens[s]) & ~((s == 0) & (p == 7))[:, None]).reshape(-1)
            K = keys[s, p, h].double().reshape(-1, d)[ok]
            V = vals[s, p, h].double().reshape(-1, d)[ok]
            use = (msk[s, h, :k][None] < taus[:, None]) | (taus == t)[:, None]
            use = use.repeat_interleave(P, 1)[:, ok]
            Q = q[s, :, h * G:(h + 1) * G].double()
            x = (Q @ K.t()) / math.sqrt(d)
            x = x.masked_fill(~use[:, None], -math.inf)
            ref_z = torch.logsumexp(x, 2)
            w = torch.exp(x - torch.where(torch.isfinite(ref_z), ref_z, 0.0)[..., None])
            ref_o = w @ V
            got_o, got_z = o[s, :, h * G:(h + 1) * G], z[s, :, h * G:(h + 1) * G]
            fin = torch.isfinite(ref_z)
            assert torch.equal(fin, torch.isfinite(got_z))
            # weights to 2^-17 (bf16 upper part + remainder), sums in fp32
            bound = 2.0 ** -16 * (w @ V.abs()) + 1e-6
            assert ((got_o - ref_o).abs() <= bound).all()
            assert (got_z[fin] - ref_z[fin]).abs().max() <= 1e-5


# a NaN key reaches every row that uses its page, and no other row
@pytest.mark.parametrize("hk", [2, 128])
@pytest.mark.parametrize("W,G", [(3, 5), (10, 8), (64, 4)])
def test_nan_key_reaches_the_rows_that_use_it(W, G, hk):
    from paper_2508_09001_amd import binding as B
    P, pages, t, bad = 16, 33, 200, 5
    lay = _layer(batch=1, num_kv_heads=hk, group=G, window=W, budget=pages * P, max_pages=pages)
    assert hk == 2 or B.retro_attend_plan(lay.dims, False)[0] == TILES[W, G]
    g = torch.Generator().manual_seed(W)
    keys = torch.randn(pages, hk, P, 128, generator=g)
    vals = torch.randn(pages, hk, P, 128, generator=g).bfloat16()
    keys[bad, :, 3, 7] = float("nan")
    lay.k_cache.copy_(keys.bfloat16())
    lay.v_cache.copy_(vals.transpose(2, 3))
    lay.seq_lens.fill_(pages * P)
    lay.num_selected.fill_(pages)
    lay.selected.copy_(torch.arange(pages, dtype=torch.int32).expand(1, hk, pages))
    msk = torch.full((1, hk, pages), -1, dtype=torch.int32)
    msk[:, :, bad] = t - W // 2 - 1          # half of the past rows may use it
    lay.mask.copy_(msk)
    q = torch.randn(1, W + 1, hk * G, 128, generator=g).bfloat16()
    print(f"[nan] hk={hk} W={W} G={G}", flush=True)
    lay.attend(t, q.cuda())
    torch.cuda.synchronize()
    o = lay.o_part.cpu().double()[0]
    good = [p for p in range(pages) if p != bad]
    for r in range(W + 1):
        if r == W or t - W + r > t - W // 2 - 1:
            assert torch.isnan(o[r]).all()
            continue
        for h in (0, hk - 1):
            K = keys[good, h].bfloat16().double().reshape(-1, 128)
            V = vals[good, h].double().reshape(-1, 128)
            w = torch.softmax(q[0, r, h * G:(h + 1) * G].double() @ K.t() / math.sqrt(128), 1)
            bound = 2.0 ** -16 * (w @ V.abs()) + 1e-6   # as above
            assert ((o[r, h * G:(h + 1) * G] - w @ V).abs() <= bound).all()


# table lengths around the stripes of the selection (512 pages each: 2, 5, 6, 9, 12)
# and past the last one; path "step": in front of the attention, "select": in the
# score launch (small tables) or a launch of its own, "launch": that launch, whatever
# the table (a step with the flag that asks for it)
@pytest.mark.parametrize("mp", [33, 512, 513, 1024, 1025, 2561, 3072, 3073, 4608, 4700, 6144, 6145])
@pytest.mark.parametrize("path", ["select", "step", "launch"])
def test_selection_matches_sorted_scores(mp, path):
    P, B, t = 16, 48 * 16, 9
    lay = _layer(batch=2, num_kv_heads=3, group=2, budget=B, window=0, max_pages=mp,
                 flags=2 if path == "launch" else 1)
    g = torch.Generator().manual_seed(mp)
    lens = torch.tensor([mp * P - 1, (mp * P) // 3])
    dig = torch.randn(2, 3, mp, 2, 128, generator=g).sort(dim=3).values
    if mp > 100:                             # equal scores: ties go to the lower page
        dig[:, 1, 50:mp - 40] = dig[:, 1, 50:51]
    lay.digest.copy_(dig)
    lay.seq_lens.copy_(lens)
    A = torch.randint(-1, t, (2, 3, mp), generator=g).int()
    lay.last_loaded.copy_(A)
    q = torch.randn(2, 1, 6, 128, generator=g).bfloat16().cuda()
    kv = torch.randn(2, 3, 128, generator=g).bfloat16().cuda()
    print(f"[select] {mp} pages, {path}", flush=True)
    if path == "select":
        lay.select(t, q[:, 0])
    else:
        lay.step(t, q, kv, kv)
        lens = lens + 1
    torch.cuda.synchronize()
    sc, sel, msk = lay.scores().cpu(), lay.selected.cpu(), lay.mask.cpu()
    new_a = lay.last_loaded.cpu()
    for s in range(2):
        n = min(-(-int(lens[s]) // P), mp)
        k = min(B // P, n)
        for h in range(3):
            want = sc[s, h, :n].sort(descending=True, stable=True).indices[:k].sort().values
            a = A[s, h].clone()
            if path != "select":
                a[(int(lens[s]) - 1) // P] = t - 1
            assert int(lay.num_selected[s, h]) == k
            assert torch.equal(sel[s, h, :k].long(), want)
            assert torch.equal(msk[s, h, :k], a[want])
            assert (sel[s, h, k:] == -1).all() and (msk[s, h, k:] == -1).all()
            a[want] = t
            assert torch.equal(new_a[s, h], a)
