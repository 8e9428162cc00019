"""GPU tests of how the interpolation spreads its points over workgroups: eighths
of the workgroups of 256 points, one eighth to an XCD, at counts where an eighth
is empty, partial or one workgroup longer, and where a workgroup takes more than
one turn.  A point's result depends on the point alone, so every count must give
the bits that the same points give in another order."""
import numpy as np
import pytest
import torch

from paper_2604_11008_amd import gen, pm

pytestmark = pytest.mark.gpu
L = gen.TWO_PI


@pytest.mark.parametrize("n", [0, 1, 255, 257, 7 * 256, 8 * 256 + 1, 9 * 256, 70 * 256 - 3,
                               65536 * 256 + 8 * 256 + 77])
def test_any_count_of_points(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[test] {n} points", flush=True)
    g = torch.Generator("cuda").manual_seed(5)
    s = (8, 6, 4)
    for ilv in (False, True):
        for ft in (torch.float64, torch.float32):
            u = [torch.randn(s[0] * s[1] * s[2], generator=g, device="cuda",
                             dtype=torch.float64).to(ft) for _ in range(3)]
            f = pm.DeviceField(torch.stack(u, dim=1) if ilv else u, s, 0, L, interleaved=ilv)
            X = torch.rand(3, n, generator=g, device="cuda", dtype=torch.float64) * L
            ctx = pm.Context(1, 1, 1)
            U = ctx.interp(f, X)
            V = ctx.interp(f, X.flip(1).contiguous()).flip(1)
            assert U.shape == (3, n) and U.dtype == ft
            assert torch.equal(U, V)
            assert n == 0 or bool((U != 0).all(0).any())
            assert ctx.get_status() == 0
            if n:       # the last point by itself
                W = ctx.interp(f, X[:, -1:].contiguous())
                np.testing.assert_array_equal(W.cpu().numpy(), U[:, -1:].cpu().numpy())
