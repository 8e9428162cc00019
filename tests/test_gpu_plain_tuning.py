"""GPU test that the plain path's scan and compaction run in the shape that
pm_get_tuning reports, a tuned one or their defaults, in pools on both sides of
the extents that change the fused step's default: the tiles that a call lays out
(a header word of the workspace) are those of the shape, the reported shape can
be set again, and the records stay bitwise the same."""
import numpy as np
import pytest
import torch

from gpu_cases import Case, assert_same_device_pools, say
from paper_2604_11008_amd import pm

pytestmark = pytest.mark.gpu
HDR_TILES = 2


@pytest.mark.parametrize("extent", [0, 1 << 20, 1 << 22])
def test_the_reported_shape_is_the_one_launched(extent):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[test] plain path's shapes, extent {extent}")
    c = Case("C2S", 30000, 32, (2, 2, 2), face=0.3, edge=0.2, corner=0.2, slack=0.3, extra=512)
    pin = pm.DevicePool.from_host(c.host, size=max(extent, c.pin().size))
    ctx = c.ctx(pin, c.send())
    ctx.interp_advance(c.field, pin, c.params)
    words = ctx.workspace.view(torch.int32)

    def launched():
        torch.cuda.synchronize()
        wg, items = ctx.get_tuning()[:2]
        assert (wg, items) in pm.SHAPES
        tiles = int((-(-np.asarray(c.host.count) // (wg * items))).sum())
        assert int(words[HDR_TILES]) == tiles, (wg, items)
        return wg, items

    ref = None
    for tuned in [(0, 0)] + pm.SHAPES:
        for bpc, xb in ((0, 0), (1, 2)):
            ctx.set_tuning(*tuned, bpc, xb)
            send, out = c.send(), c.pout(pin.size)
            ctx.classify_scan_pack(c.dc, pin, send)
            scan = launched()
            ctx.compact_append(c.dc, pin, send, out)
            move = launched()
            assert tuned == (0, 0) or scan == move == tuned
            ctx.set_tuning(*ctx.get_tuning())
            assert ctx.get_status() == 0
            ref = ref or (out, send)
            assert_same_device_pools(out, ref[0], c.dc.nsub, f"out {tuned}")
            assert_same_device_pools(send, ref[1], c.dc.nsub * 27, f"send {tuned}")
