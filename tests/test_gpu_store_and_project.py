"""Prompt storage and the fp32 projections at the edges of their shapes.

``retro_prefill_kv``: chunks that start and end inside pages, sources and caches that
are not 16-byte aligned, slots outside the chunk left as they are; bytes equal
to a plain rearrangement.  ``retro_project_f32``: the documented chain of fused
multiply-adds, bit for bit, at rows, columns, depths and alignments on both
sides of the kernel's tiles.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("P,d", [(16, 128), (32, 128), (16, 64), (32, 64)])
@pytest.mark.parametrize("off", [0, 1])
def test_prefill_chunks(dtype, P, d, off):
    from paper_2508_09001_amd import binding as B
    from paper_2508_09001_amd.layer import RetroLayer
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    hk, mp = 3, 12
    lay = RetroLayer(batch=2, num_kv_heads=hk, group=2, head_dim=d, page_size=P, budget=P, window=0,
                     max_pages=mp, dtype=dtype, page_table=torch.randperm(2 * mp).view(2, mp))
    g = torch.Generator().manual_seed(P + d + off)
    lay.k_cache.fill_(7.0)      # what was in the pool before
    lay.v_cache.fill_(9.0)
    kc, vc = lay.k_cache.cpu(), lay.v_cache.cpu()
    table = lay.page_table.cpu().long()
    at = [0, 0]
    keys = [torch.zeros(0, hk, d, dtype=td) for _ in range(2)]
    print(f"[prefill] {dtype} P={P} d={d} offset {off}", flush=True)
    for seq, n in [(0, 1), (1, 3 * P + 5), (0, P - 2), (0, 1), (0, 2 * P), (1, 3), (0, P // 2 + 1),
                   (1, 2 * P + 8), (0, 1), (0, 5)]:
        k, v = torch.randn(n, hk, d, generator=g).to(td), torch.randn(n, hk, d, generator=g).to(td)
        buf = [torch.empty(n * hk * d + 8, dtype=td, device="cuda") for _ in range(2)]
        src = [x[off:off + n * hk * d] for x in buf]
        src[0].copy_(k.reshape(-1))
        src[1].copy_(v.reshape(-1))
        B.retro_prefill_kv(lay.dims, lay.cache, seq, at[seq], n, src[0], src[1])
        pos = torch.arange(at[seq], at[seq] + n)
        kc[table[seq][pos // P], :, pos % P] = k
        vc[table[seq][pos // P], :, :, pos % P] = v
        keys[seq] = torch.cat([keys[seq], k])
        at[seq] += n
        torch.cuda.synchronize()
        assert torch.equal(lay.k_cache.cpu(), kc)
        assert torch.equal(lay.v_cache.cpu(), vc)
    assert lay.seq_lens.tolist() == at
    for s in range(2):
        for p in range(-(-at[s] // P)):
            page = keys[s][p * P:(p + 1) * P]
            dg = lay.digest[s, :, p].cpu()
            assert torch.equal(dg[:, 0], page.amin(0)) and torch.equal(dg[:, 1], page.amax(0))


# rows around the blocks of 8 and 32, columns around 16, depths around the slab of
# 256 and the four of a trip; off 1: w not 16-byte aligned
@pytest.mark.parametrize("rows,K,n,off", [(1, 1, 1, 0), (5, 255, 16, 0), (8, 256, 20, 0),
                                          (9, 257, 31, 0), (32, 1024, 48, 1), (33, 1027, 32, 0),
                                          (70, 2049, 17, 1), (3, 1280, 64, 1),
                                          # more blocks of eight rows than compute units
                                          (9, 257, 2201, 0), (33, 300, 1000, 0),
                                          (70, 1027, 500, 1)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_project_f32_is_the_documented_chain(rows, K, n, off, accumulate):
    from paper_2508_09001_amd import binding as B
    rng = np.random.default_rng(rows * K + n)
    x = rng.standard_normal((rows, K), dtype=np.float32)
    w = rng.standard_normal((K, n), dtype=np.float32)
    y0 = rng.standard_normal((rows, n), dtype=np.float32)
    # a fused multiply-add through 64-bit mantissas: the product is exact, and the
    # sum's second rounding differs from one rounding in about one case of 2^40
    acc = np.zeros((rows, n), np.float32)
    for i in range(K):
        acc = (x[:, i:i + 1].astype(np.longdouble) * w[i].astype(np.longdouble) + acc).astype(np.float32)
    want = y0 + acc if accumulate else acc
    buf = torch.empty(K * n + 4, device="cuda")
    wd = buf[off:off + K * n]
    wd.copy_(torch.from_numpy(w).reshape(-1))
    y = torch.from_numpy(y0).cuda()
    print(f"[f32] rows={rows} K={K} n={n} offset {off}", flush=True)
    B.retro_project_f32(torch.from_numpy(x).cuda(), rows, K, wd, n, y, accumulate=accumulate)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), want)


# runs of 1 token to more than the sequence holds, inside a page and across pages
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("P,d", [(16, 128), (32, 64)])
@pytest.mark.parametrize("n", [1, 7, 16, 33, 70])
def test_update_kv_runs(dtype, P, d, n):
    from paper_2508_09001_amd.layer import RetroLayer
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    hk, mp, lens = 3, 8, [1, 5 * P, 2 * P + 3, 40]
    lay = RetroLayer(batch=4, num_kv_heads=hk, group=2, head_dim=d, page_size=P, budget=P, window=0,
                     max_pages=mp, dtype=dtype, page_table=torch.randperm(4 * mp).view(4, mp))
    g = torch.Generator().manual_seed(n + P)

    def rand(*s):
        return torch.randn(*s, generator=g).to(td)

    keys, vals = [rand(x, hk, d) for x in lens], [rand(x, hk, d) for x in lens]
    for s in range(4):
        lay.prefill(s, keys[s], vals[s])
    ku, vu = rand(4, n, hk, d), rand(4, n, hk, d)
    print(f"[update] {dtype} P={P} d={d} n={n}", flush=True)
    lay.update_kv(ku, vu)
    torch.cuda.synchronize()
    table, kc, vc = lay.page_table.cpu().long(), lay.k_cache.cpu(), lay.v_cache.cpu()
    for s, length in enumerate(lens):
        m = min(n, length)
        k = torch.cat([keys[s][:length - m], ku[s, n - m:]])
        v = torch.cat([vals[s][:length - m], vu[s, n - m:]])
        pos = torch.arange(length)
        assert torch.equal(kc[table[s][pos // P], :, pos % P], k)
        assert torch.equal(vc[table[s][pos // P], :, :, pos % P], v)
        for p in range(-(-length // P)):
            dg = lay.digest[s, :, p].cpu()
            page = k[p * P:(p + 1) * P]
            assert torch.equal(dg[:, 0], page.amin(0)) and torch.equal(dg[:, 1], page.amax(0))
    assert lay.seq_lens.tolist() == lens
