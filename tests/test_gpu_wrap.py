"""GPU tests of the stencil corners where they wrap or leave the grid: points in
the first and last cells of every axis (whole waves of them, and single lanes
among others), over the periodic images, on grids down to two cells, split and
interleaved, float64 and float32; and points beyond the images, NaN and
infinities, which raise PM_F_HALO (but NaN) and are moved to the nearest stored
corner.  Tolerance: seven lerps of values up to max|u| with a fraction of the
position's rounding times the grid's steepest slope: 64 ulps of max|u|."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu
L = gen.TWO_PI


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def interp(u, n, halo, X, ilv):
    f = pm.DeviceField(torch.stack(u, dim=1) if ilv else u, n, halo, L, interleaved=ilv)
    ctx = pm.Context(1, 1, 1)
    U = ctx.interp(f, X)
    return U.cpu().numpy(), ctx.get_status()


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("halo", [0, 1])
@pytest.mark.parametrize("n", [(2, 3, 2), (5, 2, 17), (33, 16, 4)])
def test_corners_at_the_seams(n, halo, mixed):
    print(f"[test] seams n={n} halo={halo} mixed={mixed}", flush=True)
    g = np.random.default_rng(sum(n) + halo)
    m = 64 * 6 + 5
    X = g.uniform(0.0, L, (3, m))
    for a in range(3):
        cell = L / n[a]
        X[a, 64 * a:64 * a + 64] = L - 0.4 * cell * g.uniform(0, 1, 64)     # a wave of wraps
        X[a, 192 + 64 * (a % 2):256 + 64 * (a % 2):9] = 0.3 * cell          # some lanes
        if not halo:
            X[a, 320 + a:m:3] += g.choice([-L, L], len(range(320 + a, m, 3)))
    ft = np.float32 if mixed else np.float64
    uh = [g.standard_normal((n[2], n[1], n[0])).astype(ft) for _ in range(3)]
    st = [np.ascontiguousarray(gen.with_halo(u) if halo else u).reshape(-1) for u in uh]
    u = [torch.from_numpy(a).cuda() for a in st]
    Xd = torch.from_numpy(X).cuda()
    U, fl = interp(u, n, halo, Xd, False)
    V, fl2 = interp(u, n, halo, Xd, True)
    # a periodic field is stored for a box to either side: -n <= s < 2n
    sn = X * (np.array(n) / L)[:, None] - 0.5
    off = (np.zeros(m, bool) if halo else
           ((sn < -np.array(n)[:, None]) | (sn >= 2 * np.array(n)[:, None])).any(0))
    want = pm.HALO if off.any() else 0
    assert fl == want and fl2 == want, (fl, fl2, want)
    np.testing.assert_array_equal(U, V)
    ref, _ = oracle.interp(oracle.Field([a.astype(np.float64) for a in st], n, halo,
                                        (L, L, L)), X)
    umax = max(np.abs(a).max() for a in st)
    # the position's rounding: a few ulps of s = X n / L - 1/2 times the slope
    eps = np.finfo(ft).eps
    slack = 64 * eps * umax + 16 * np.finfo(np.float64).eps * 2 * max(n) * 2 * umax
    err = np.abs(U - ref)[:, ~off].max()
    assert err <= slack, err


@pytest.mark.parametrize("halo", [0, 1])
def test_points_off_the_grid(halo):
    print(f"[test] off the grid halo={halo}", flush=True)
    n = (8, 4, 6)
    g = np.random.default_rng(7)
    st = [n[a] + 2 * halo for a in range(3)]
    u = [torch.from_numpy(g.standard_normal(st[0] * st[1] * st[2])).cuda() for _ in range(3)]
    inside = g.uniform(0.2, 6.0, (3, 64))
    # lane 5: no flag for a NaN, whatever it reads; the others far off on one axis
    X = inside.copy()
    X[1, 5] = np.nan
    U, fl = interp(u, n, halo, torch.from_numpy(X).cuda(), False)
    V, fl2 = interp(u, n, halo, torch.from_numpy(X).cuda(), True)
    assert fl == 0 and fl2 == 0
    assert np.isnan(U[:, 5]).all() and np.isnan(V[:, 5]).all()
    np.testing.assert_array_equal(np.delete(U, 5, 1), np.delete(V, 5, 1))
    for a in range(3):
        for far in (-2.0 * L, 3.0 * L, 1e300, -1e300, np.inf):
            X = inside.copy()
            X[a, 17] = far
            U, fl = interp(u, n, halo, torch.from_numpy(X).cuda(), False)
            V, fl2 = interp(u, n, halo, torch.from_numpy(X).cuda(), True)
            assert fl == pm.HALO and fl2 == pm.HALO, (a, far, fl, fl2)
            np.testing.assert_array_equal(U, V)
