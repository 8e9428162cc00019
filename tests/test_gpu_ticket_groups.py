"""GPU test of the tile order by ticket groups on few tiles: blocks that give all
tiles to one group, to some, or one to each, in grids of more and of fewer
workgroups than tiles.  Every setting must give bitwise the records of the one
counter, through the step, per-stage migration and the plain path."""
import pytest
import torch

from gpu_cases import Case, assert_same_device_pools, say
from paper_2604_11008_amd import pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npart", [200, 3000, 20000, 140000])
def test_groups_on_few_tiles(npart):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[test] ticket groups, {npart} records")
    c = Case("C2S", npart, 32, (2, 1, 2), face=0.3, edge=0.2, corner=0.2, slack=0.3, extra=512)
    c.params = pm.Params(0.015, c.g)
    pin = c.pin()
    ctx = c.ctx(pin, c.send())
    ref = None
    for xb in (0, 1, 2, 7, 64, 65536):
        for bpc in (0, 1, 8):
            say(f"  xcd_block={xb} blocks_per_cu={bpc}")
            ctx.set_tuning(256, 1, bpc, xb)
            send, out, send2, out2 = c.send(), c.pout(pin.size), c.send(), c.pout(pin.size)
            send3, out3 = c.send(), c.pout(pin.size)
            ctx.step(c.field, c.dc, pin, out, send, c.params)
            mid = pm.DeviceStagePool.empty(c.host.base, c.host.cap, vdtype=c.vdt, size=pin.size)
            mids = pm.DeviceStagePool.empty(c.sb, c.sc, vdtype=c.vdt, size=send.size)
            ctx.step_staged(c.field, c.dc, pin, mid, mids, out2, send2, c.params)
            plain = c.pin()
            ctx.interp_advance(c.field, plain, c.params)
            ctx.classify_scan_pack(c.dc, plain, send3)
            ctx.compact_append(c.dc, plain, send3, out3)
            assert ctx.get_status() == 0
            got = (out, send, out2, send2, out3, send3)
            ref = ref or got
            for k, (a, b) in enumerate(zip(got, ref)):
                assert_same_device_pools(a, b, c.dc.nsub * (27 if k % 2 else 1), f"output {k}")
