"""GPU test of how the interpolation deals its points to the XCDs, in chunks of 16
workgroups of 256: counts on both sides of a workgroup, a chunk and a round of
eight chunks, split and interleaved, with fewer points than cells and with more.
Against the oracle; tolerance: the rounding of seven lerps of values up to
max|u|, 64 ulps of it, and of the position times the grid's slope."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu
L = gen.TWO_PI


@pytest.mark.parametrize("cells", [4, 40])
@pytest.mark.parametrize("n", [16 * 256 - 1, 16 * 256, 16 * 256 + 1, 128 * 256 - 255, 128 * 256,
                               128 * 256 + 1, 144 * 256 + 3])
def test_chunks(n, cells):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[test] {n} points, {cells}^3 cells", flush=True)
    g = np.random.default_rng(n)
    u = [g.standard_normal(cells ** 3) for _ in range(3)]
    X = g.uniform(0.0, L, (3, n))
    ref, f0 = oracle.interp(oracle.Field(u, cells, 0, L), X)
    assert f0 == 0
    eps, umax = np.finfo(np.float64).eps, max(np.abs(a).max() for a in u)
    ud = [torch.from_numpy(a).cuda() for a in u]
    ctx = pm.Context(1, 1, 1)
    for ilv in (False, True):
        f = pm.DeviceField(torch.stack(ud, dim=1) if ilv else ud, cells, 0, L, interleaved=ilv)
        U = ctx.interp(f, torch.from_numpy(X).cuda()).cpu().numpy()
        assert ctx.get_status() == 0
        assert np.abs(U - ref).max() <= (64 + 64 * cells) * eps * umax


def test_sparse_points_in_eighths():
    """Few points a cell and many of them: an eighth of the workgroups to an XCD.
    The same points in another order, and some by themselves, give the same bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, cells = (1 << 22) + 3 * 256 + 11, 384
    print(f"[test] {n} points, {cells}^3 cells", flush=True)
    g = torch.Generator("cuda").manual_seed(3)
    u = [torch.randn(cells ** 3, generator=g, device="cuda", dtype=torch.float32)
         for _ in range(3)]
    X = torch.rand(3, n, generator=g, device="cuda", dtype=torch.float64) * L
    ctx = pm.Context(1, 1, 1)
    for stag in (False, True):
        f = pm.DeviceField(u, cells, 0, L, stagger=stag)
        U = ctx.interp(f, X)
        assert torch.equal(U, ctx.interp(f, X.flip(1).contiguous()).flip(1))
        k = torch.arange(0, n, 4099, device="cuda")
        assert torch.equal(U[:, k], ctx.interp(f, X[:, k].contiguous()))
        assert torch.equal(U[:, -300:], ctx.interp(f, X[:, -300:].contiguous()))
        assert bool((U != 0).all())
    assert ctx.get_status() == 0
