"""GPU tests of the cell re-sort at the sizes where its tiles and keys change:
segments of a tile's 4096 records and one more or less, near-empty ones, pools
in one cell (every digit the same), keys of 32 bits with 8- and 9-bit digits and
of 64 bits (more than 1024 cells an axis).  Against the definition written out
with numpy; whole records are moved, so every comparison is exact."""
import numpy as np
import pytest
import torch

from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,counts,spread,mixed", [
    ((64, 64, 64), (4095, 4096, 4097, 1, 0, 8193), 1.0, False),
    ((256, 256, 256), (70000, 3, 4096 * 5), 1.0, False),   # 25-bit keys: 9-bit digits
    ((256, 256, 256), (30011,), 0.003, True),              # a few cells
    ((512, 300, 7), (20000, 511, 513), 1.0, True),         # 28-bit keys
    ((1024, 16, 1000), (9000, 12000), 1.0, False),         # 31-bit keys
    ((1030, 12, 2050), (5000, 9001, 64), 1.0, False),      # 64-bit keys
])
def test_sort_tiles_and_key_widths(n, counts, spread, mixed):
    print(f"[test] re-sort n={n} counts={counts} spread={spread} mixed={mixed}", flush=True)
    g = np.random.default_rng(len(counts) + n[0])
    L = gen.TWO_PI
    base, cap = gen.layout(np.array(counts), slack=0.1, extra=7, align=1)
    size = int((base + cap).max())
    vd = np.float32 if mixed else np.float64
    pool = gen.empty_pool(base, cap, vd)
    pool.x[:] = gen.into_box(1.0 + spread * g.uniform(0.0, L, (3, size)))
    pool.v[:] = g.standard_normal((3, size))
    pool.tau[:] = g.uniform(0.1, 1.0, size)
    pool.id[:] = g.permutation(size).astype(np.uint64)
    pool.count[:] = counts
    ft = torch.float32 if mixed else torch.float64
    field = pm.DeviceField(torch.zeros((n[0] * n[1] * n[2], 3), dtype=ft, device="cuda"), n, 0,
                           L, interleaved=True)
    pin = pm.DevicePool.from_host(pool)
    pout = pm.DevicePool.empty(base, cap, vdtype=ft, size=pin.size)
    ctx = pm.Context(pin.size, 1, len(counts))
    for _ in range(2):  # a second sort finds the first one's workspace
        ctx.sort(field, pin, pout)
    assert ctx.get_status() == 0
    out = pout.to_host()
    np.testing.assert_array_equal(out.count, pool.count)
    for b, c in zip(base, counts):
        x = pool.x[:, b:b + c]
        cell = [np.clip(np.floor(x[a] * (n[a] / L)).astype(np.int64), 0, n[a] - 1)
                for a in range(3)]
        # gen.cell_key over 20 bits an axis (its own 11 hold grids up to 2048)
        key = gen.morton3(cell[0] >> 1, cell[1], cell[2], bits=20) * 2 + (cell[0] & 1)
        src = b + np.argsort(key, kind="stable")
        for name in ("x", "v", "tau", "id"):
            np.testing.assert_array_equal(getattr(out, name)[..., b:b + c],
                                          getattr(pool, name)[..., src], err_msg=name)
        # nothing past the segment's records
        assert not out.id[b + c:b + cap[list(base).index(b)]].any()
