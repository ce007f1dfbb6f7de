"""More pairs than 32 bits can count: a total of 2^32 + 8,192, which would look
like 8,192 if it wrapped, is refused or reported, and no tile has a list."""
import numpy as np
import pytest
import torch

import synth
from tests import _gpu as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("capacity", [0, 1 << 27])
def test_a_total_past_32_bits_is_an_overflow(capacity):
    from paper_2410_04974_amd import SixDGSError, _lib
    cams = [synth.default_camera(512, 512)] * 8
    n = 2**19 + 1  # entries of 1,024 tiles each, 16 patches: 67M items, which fit the fixed capacity
    E = n * len(cams)
    full = lambda x: torch.full((E,), x, device=G.DEV)  # noqa: E731
    rec = [full(256.0), full(256.0), full(400.0), full(400.0), full(2.0),
           torch.ones(E, dtype=torch.int32, device=G.DEV)]
    r = G.renderer(pair_capacity=capacity)
    with pytest.raises(SixDGSError) as e:
        r.ctx.bin(n, cams, *rec)
        assert capacity, "a growing context refuses the call itself"
        assert not r.ctx.export(_lib.EXPORT_RANGES).any()
        r.ctx.check()
    print(capacity, e.value, flush=True)
    assert e.value.status == _lib.ERR_CAPACITY
    # and the next call of the same context is a plain one: pixels 15 to 25 each way, four tiles
    u = torch.full((1,), 20.0, device=G.DEV)
    r.ctx.bin(1, cams[:1], u, u, u / 4, u / 4, u, torch.ones(1, dtype=torch.int32, device=G.DEV))
    r.ctx.check()
    assert r.ctx.sizes()["pairs"] == 4 and np.array_equal(r.ctx.export(_lib.EXPORT_VALUES), [0] * 4)
