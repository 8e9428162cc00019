"""GPU tests of the plain path's scan and compaction where their tiles change:
pools on both sides of the extents that pick 256, 1024 or 4096 records a tile,
segments ending in, before and after a run of 64 records, launched over
sub-ranges too.  The oracle's sequential partition and append of the same
records must be matched bit for bit (nothing is computed but copies and the
periodic shift)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_cases import compare_pools
from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("counts,extent,mixed,split", [
    ((63, 64, 65, 1, 0, 255, 256, 257), 0, False, False),        # 256 a tile
    ((1023, 1024, 1025, 64, 5000, 0, 4097, 129), 1 << 20, True, True),      # 1024
    ((4095, 4096, 4097, 8192, 1, 0, 20000, 12289), 1 << 22, False, True),   # 4096
])
def test_exchange_tiles(counts, extent, mixed, split):
    print(f"[test] exchange counts={counts} extent={extent} mixed={mixed}", flush=True)
    g = np.random.default_rng(len(counts) + extent)
    L, p = gen.TWO_PI, (2, 2, 2)
    bnds = gen.bounds(p, L)
    cell = L / 64
    base, cap = gen.layout(np.array(counts), slack=0.5, extra=4000)
    vd = np.float32 if mixed else np.float64
    pool = gen.empty_pool(base, cap, vd)
    for s, (b, c) in enumerate(zip(base, counts)):
        k = (s % 2, (s // 2) % 2, s // 4)
        for a in range(3):
            # in the owner's box or up to a cell outside of it
            lo, hi = bnds[a][k[a]] - cell, bnds[a][k[a] + 1] + cell
            pool.x[a, b:b + c] = g.uniform(lo, hi, c)
    pool.v[:] = g.standard_normal(pool.v.shape)
    pool.tau[:] = g.uniform(0.1, 1.0, pool.size)
    pool.id[:] = g.permutation(pool.size).astype(np.uint64)
    pool.count[:] = counts
    sb, sc = gen.send_layout(counts, face=0.2, edge=0.1, corner=0.1)
    ft = torch.float32 if mixed else torch.float64
    pin = pm.DevicePool.from_host(pool, size=max(extent, pool.size))
    pout = pm.DevicePool.empty(base, cap, vdtype=ft, size=pin.size)
    send = pm.DevicePool.empty(sb, sc, vdtype=ft)
    dc = pm.Decomp(p, bnds)
    ctx = pm.Context(pin.size, send.size, dc.nsub)
    ranges = [(0, 3), (3, 1), (4, 4)] if split else [(0, 8)]
    if split:
        # the stayers' counts live until the next classify call: one call a pack
        ctx.classify_scan_pack(dc, pin, send)
        for f, c in ranges:
            ctx.compact_append(dc, pin, send, pout, f, c)
    else:
        for _ in range(2):
            ctx.classify_scan_pack(dc, pin, send)
            ctx.compact_append(dc, pin, send, pout)
    assert ctx.get_status() == 0
    rout = gen.empty_pool(base, cap, vd)
    rsend = gen.empty_pool(sb, sc, vd)
    stay, f1 = oracle.partition(oracle.Decomp(p, bnds), pool, rout, rsend)
    f2 = oracle.append(oracle.Decomp(p, bnds), rsend, stay, rout)
    assert f1 == 0 and f2 == 0
    assert rsend.count.sum() > 0
    compare_pools(send.to_host(), rsend, dc.nsub * 27, L, cell, exact=True, what="send")
    compare_pools(pout.to_host(), rout, dc.nsub, L, cell, exact=True, what="out")


@pytest.mark.parametrize("extent", [0, 1 << 20, 1 << 22])
def test_records_changed_after_the_classification(extent):
    """pm_compact_append moves what pm_classify_scan_pack found to stay, with the
    values that the records hold by then; runs of 1, 2, 3 and 64 records too."""
    print(f"[test] changed records extent={extent}", flush=True)
    counts = (1, 2, 3, 65, 66, 67, 4160, 64)
    g = np.random.default_rng(3)
    L, p = gen.TWO_PI, (2, 2, 2)
    bnds = gen.bounds(p, L)
    base, cap = gen.layout(np.array(counts), slack=0.5, extra=4000)
    pool = gen.empty_pool(base, cap, np.float64)
    for s, (b, c) in enumerate(zip(base, counts)):
        k = (s % 2, (s // 2) % 2, s // 4)
        for a in range(3):
            lo, hi = bnds[a][k[a]], bnds[a][k[a] + 1]
            pool.x[a, b:b + c] = g.uniform(lo - 0.5, hi + 0.5, c)
    pool.v[:] = g.standard_normal(pool.v.shape)
    pool.tau[:] = g.uniform(0.1, 1.0, pool.size)
    pool.id[:] = np.arange(pool.size, dtype=np.uint64)
    pool.count[:] = counts
    sb, sc = gen.send_layout(counts, face=1.0, edge=1.0, corner=1.0)
    pin = pm.DevicePool.from_host(pool, size=max(extent, pool.size))
    pout = pm.DevicePool.empty(base, cap, vdtype=torch.float64, size=pin.size)
    send = pm.DevicePool.empty(sb, sc, vdtype=torch.float64)
    dc = pm.Decomp(p, bnds)
    ctx = pm.Context(pin.size, send.size, dc.nsub)
    ctx.classify_scan_pack(dc, pin, send)
    for a in range(3):
        pin.x[a].copy_(pin.x[a].flip(0))
    ctx.compact_append(dc, pin, send, pout)
    assert ctx.get_status() == 0
    rout = gen.empty_pool(base, cap, np.float64)
    rsend = gen.empty_pool(sb, sc, np.float64)
    stay, f1 = oracle.partition(oracle.Decomp(p, bnds), pool, rout, rsend)
    f2 = oracle.append(oracle.Decomp(p, bnds), rsend, stay, rout)
    assert f1 == 0 and f2 == 0 and rsend.count.sum() > 0
    x = np.stack([pin.x[a].cpu().numpy() for a in range(3)])
    got = pout.to_host()
    np.testing.assert_array_equal(got.count, rout.count)
    for s, b in enumerate(base):
        n = int(stay[s])
        ids = rout.id[b:b + rout.count[s]]
        np.testing.assert_array_equal(got.id[b:b + rout.count[s]], ids)
        np.testing.assert_array_equal(got.x[:, b:b + n], x[:, ids[:n].astype(np.int64)])
        np.testing.assert_array_equal(got.x[:, b + n:b + rout.count[s]],
                                      rout.x[:, b + n:b + rout.count[s]])
