"""The debug mode takes the records that the normal mode takes, NaN coordinates
of a caller's binning among them, and leaves the same lists."""
import numpy as np
import pytest
import torch

import synth
from tests import _gpu as G
from tests.test_gpu_parity import _random_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["u", "v", "ex", "u and v"])
def test_undefined_coordinates_in_the_debug_mode(which):
    from paper_2410_04974_amd import _lib
    cams, n = [synth.default_camera(200, 150), synth.default_camera(90, 400)], 500
    rec = dict(zip(("u", "v", "ex", "ey", "depth", "alive"), _random_records(n, cams, seed=6, ext=20.0)))
    for name in which.split(" and "):
        rec[name][::9] = np.nan
    out = []
    for flags in (0, _lib.FLAG_DEBUG):
        r = G.renderer(flags=flags)
        r.ctx.bin(n, cams, *(torch.from_numpy(a).to(G.DEV) for a in rec.values()))
        r.ctx.check()
        out.append([r.ctx.export(k) for k in (_lib.EXPORT_KEYS, _lib.EXPORT_VALUES, _lib.EXPORT_RANGES)])
    print(which, len(out[0][1]), flush=True)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
