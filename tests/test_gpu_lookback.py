"""GPU tests of the look-back over the tiles of a segment: segments of one tile
up to more tiles than one read of status words covers (1024), on both sides of
the 64 tiles after which counts are handed on, with leavers in every tile.  The
oracle's sequential partition and append of the device's own advanced records
must be matched bit for bit."""
import pytest
import torch

from gpu_cases import Case, lockstep_migration, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("npart,p,shape,mode", [
    (700000, (2, 1, 1), (256, 1), None),     # about 1367 tiles a segment
    (600000, (1, 1, 1), (256, 1), "mixed"),  # 2344 tiles, one segment
    (130000, (2, 2, 2), (256, 1), None),     # 63 to 65 tiles a segment
    (9000, (4, 3, 3), (256, 1), None),       # one tile a segment
    (700000, (1, 2, 1), (512, 2), None),     # about 342 tiles of 1024
])
def test_lookback_over_many_tiles(npart, p, shape, mode):
    say(f"[test] look-back {npart} {p} {shape} {mode}")
    c = Case("C2S", npart, 64, p, mode=mode, face=0.3, edge=0.15, corner=0.1, dt_scale=0.5,
             slack=0.3, extra=4000)
    pin, send = c.pin(), c.send()
    out = c.pout(pin.size)
    ctx = c.ctx(pin, send)
    ctx.set_tuning(*shape)
    for _ in range(2):
        ctx.step(c.field, c.dc, pin, out, send, c.params)
    assert ctx.get_status() == 0
    assert lockstep_migration(c, ctx, pin, out, send) > npart // 1000
