"""The tiles' lists at the edges of how they are built: patches of 8 x 8 tiles
(images of one, a little more and less), chunks of the tested entries (256 and
1,024), and the items sorted by patch in one and in two radix passes, growing
and at a fixed capacity, with the depths sorted by counting (up to 20,480
entries) and by radix passes -- against the oracle's sorted pairs, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests import _gpu as G
from tests.test_gpu_parity import _random_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,n,ext,tile", [
    ([(128, 128)], 1, 30.0, (16, 16)), ([(128, 128)], 255, 30.0, (16, 16)), ([(128, 128)], 257, 30.0, (32, 8)),
    ([(129, 127)], 1024, 30.0, (16, 16)), ([(127, 129), (16, 16), (144, 130)], 1025, 60.0, (16, 16)),
    ([(1000, 1000)], 16000, 10.0, (16, 16)), ([(1000, 1000)], 17000, 10.0, (16, 16)),  # 256 and 1,024 per workgroup
    ([(1000, 1000)], 20481, 10.0, (8, 32)), ([(1700, 40)], 20480, 25.0, (16, 16)),
    ([(512, 512)] * 16, 8500, 12.0, (16, 16)),             # sorted items, 256 patches
    ([(640, 512), (200, 500)] * 8, 12000, 12.0, (16, 16)),  # two passes
    ([(640, 512), (200, 500)] * 8, 12000, 300.0, (32, 8))])
def test_lists_bit_exact(sizes, n, ext, tile):
    from paper_2410_04974_amd import SixDGSError, _lib
    cams = [synth.default_camera(*s) for s in sizes]
    u, v, ex, ey, depth, alive = _random_records(n, cams, seed=n, ext=ext)
    ref = oracle.bin_records(u, v, ex, ey, depth, alive.astype(bool), n, cams, *tile)
    P = len(ref["keys"])
    ranges = np.where(ref["ranges"][:, :1] < ref["ranges"][:, 1:], ref["ranges"], 0)  # an empty tile has (0, 0)
    dev = [torch.from_numpy(a).to(G.DEV) for a in (u, v, ex, ey, depth, alive)]
    for cap in (0, P + 77):
        r = G.renderer(tile=tile, pair_capacity=cap)
        r.ctx.bin(n, cams, *dev)
        r.ctx.check()
        print(sizes[0], n, "pairs", P, "capacity", cap, flush=True)
        assert np.array_equal(r.ctx.export(_lib.EXPORT_KEYS), ref["keys"])
        assert np.array_equal(r.ctx.export(_lib.EXPORT_VALUES), ref["values"].astype(np.int32))
        assert np.array_equal(r.ctx.export(_lib.EXPORT_RANGES), ranges.astype(np.int32))
    if P > 1:
        small = G.renderer(tile=tile, pair_capacity=P - 1)
        small.ctx.bin(n, cams, *dev)
        assert not small.ctx.export(_lib.EXPORT_RANGES).any()
        with pytest.raises(SixDGSError) as e:
            small.ctx.check()
        assert e.value.status == _lib.ERR_CAPACITY


def test_depths_of_any_bit_pattern_are_ordered_by_counting():
    """The caller's depths may be NaN with every bit set: these entries come last
    in every tile, in entry order, and each stands where it belongs once."""
    from paper_2410_04974_amd import _lib
    cams, n = [synth.default_camera(200, 150)], 3000
    u, v, ex, ey, depth, alive = _random_records(n, cams, seed=3, ext=20.0)
    odd = np.arange(n) % 3 == 0
    depth[odd] = 1e30  # where the oracle puts them
    ref = oracle.bin_records(u, v, ex, ey, depth, alive.astype(bool), n, cams, 16, 16)
    depth.view(np.uint32)[odd] = 0xFFFFFFFF
    r = G.renderer()
    r.ctx.bin(n, cams, *(torch.from_numpy(a).to(G.DEV) for a in (u, v, ex, ey, depth, alive)))
    r.ctx.check()
    assert np.array_equal(r.ctx.export(_lib.EXPORT_VALUES), ref["values"].astype(np.int32))
