"""GPU test of waves whose stencils wrap around a periodic interleaved field:
no lane of a wave, its first, its last, some or all of them in the last cells
along x, at the first stage, at the second one only (the particle moves there)
or at both, on grids down to two cells.  Step, in-place advance, per-stage
migration and interpolation must give bitwise the split field's records, whose
wrap is each lane's own."""
import numpy as np
import pytest
import torch

from gpu_cases import assert_same_device_pools
from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu
L = gen.TWO_PI


def records(n, mixed):
    """Whole waves of each kind, and a ragged end; one cell of movement a step."""
    g = np.random.default_rng(n)
    cell = L / n
    kinds = 12
    m = 64 * kinds * 3 + 37
    X = g.uniform(0.0, L, (3, m))
    V = 0.2 * g.standard_normal((3, m))
    inner = max(n - 2, 1)                       # cells away from the wrap
    X[0] = (0.6 + g.uniform(0.0, 1.0, m) * (inner - 0.4)) * cell if n > 2 else 0.6 * cell
    lane, kind = np.arange(m) % 64, (np.arange(m) // 64) % kinds
    pick = [lane < 0, lane == 0, lane == 63, lane % 5 == 2, lane >= 0, g.random(m) < 0.02]
    near = L - 0.2 * cell * g.uniform(0.0, 1.0, m)      # wraps at stage 1
    before = L - 0.52 * cell                            # and V carries it over at stage 2
    for k in range(kinds):
        w = (kind == k) & pick[k % 6]
        X[0, w] = near[w] if k < 6 else before
        if k >= 6:
            V[0, w] = 0.3 * cell
    X[0] = np.clip(X[0], 0.0, np.nextafter(L, 0.0))
    vd = np.float32 if mixed else np.float64
    base, cap = gen.layout(np.array([m]), slack=0.1, extra=256)
    pool = gen.empty_pool(base, cap, vd)
    pool.x[:, :m], pool.v[:, :m] = X, V.astype(vd)
    pool.tau[:m] = g.uniform(0.5, 2.0, m).astype(vd)
    pool.id[:m] = np.arange(m)
    pool.count[:] = m
    return pool


@pytest.mark.parametrize("drag", ["stokes", "nonlinear"])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [2, 3, 7, 64])
def test_waves_that_wrap(n, mixed, drag):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[test] wrapping waves n={n} mixed={mixed} {drag}", flush=True)
    host = records(n, mixed)
    ft = torch.float32 if mixed else torch.float64
    g = torch.Generator("cuda").manual_seed(n)
    u = [torch.randn(n ** 3, generator=g, device="cuda", dtype=torch.float64).to(ft)
         for _ in range(3)]
    fields = (pm.DeviceField(u, n, 0, L),
              pm.DeviceField(torch.stack(u, dim=1), n, 0, L, interleaved=True))
    dc = pm.Decomp((1, 1, 1), gen.bounds((1, 1, 1), L))
    m = int(host.count[0])
    sb, sc = gen.send_layout(host.count, face=1.0, edge=0.5, corner=0.5)
    params = pm.Params(0.9, (0.0, 0.0, 0.0), drag=drag)
    res = []
    for f in fields:
        pin = pm.DevicePool.from_host(host)
        new = lambda: pm.DevicePool.empty(host.base, host.cap, vdtype=ft, size=pin.size)  # noqa: E731
        snd = lambda: pm.DevicePool.empty(sb, sc, vdtype=ft)  # noqa: E731
        out, send, out2, send2, adv = new(), snd(), new(), snd(), pm.DevicePool.from_host(host)
        ctx = pm.Context(pin.size, send.size, 1)
        U = ctx.interp(f, pin.x[:, :m].contiguous())
        ctx.step(f, dc, pin, out, send, params)
        ctx.interp_advance(f, adv, params)
        mid = pm.DeviceStagePool.empty(host.base, host.cap, vdtype=ft, size=pin.size)
        mids = pm.DeviceStagePool.empty(sb, sc, vdtype=ft, size=send.size)
        ctx.step_staged(f, dc, pin, mid, mids, out2, send2, params)
        flags = ctx.get_status()
        res.append((U, out, send, adv, out2, send2, flags))
    assert torch.equal(res[0][0], res[1][0])
    # a record that nonlinear drag throws far may be flagged, in both alike
    assert res[0][6] == res[1][6] and (res[0][6] == 0 or drag == "nonlinear")
    for k, (what, segs) in enumerate((("out", 1), ("send", 27), ("advance", 1),
                                      ("staged out", 1), ("staged send", 27)), 1):
        assert_same_device_pools(res[0][k], res[1][k], segs, what)
