"""The integer stage's scratch: the lists' table stands in the item passes'
place where it fits there (a first call pays for every byte it allocates), has
room of its own where it does not, and nothing is written past either."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from tests import _gpu as G
from tests.test_gpu_parity import _random_records

pytestmark = pytest.mark.gpu


def state_bytes(r):
    from paper_2410_04974_amd import _lib as L
    ptr, nbytes = ctypes.c_void_p(), ctypes.c_int64()
    assert L.lib().sixdgs_debug_buffer(r.ctx._h, b"sort state", ctypes.byref(ptr), ctypes.byref(nbytes)) == L.OK
    return nbytes.value


@pytest.mark.parametrize("n,size,ext,capacity,own", [
    (100000, 800, 4.0, 3_000_000, False),  # 49 patches x 98 chunks of entries: 1.2 MB of rows beside 6 MB of passes
    (16000, 1000, 2.0, 40_000, True),      # 64 patches x 63 short chunks: 1 MB beside 82 KB
])
def test_the_table_of_the_lists(n, size, ext, capacity, own):
    from paper_2410_04974_amd import _lib
    cams = [synth.default_camera(size, size)]
    rec = _random_records(n, cams, seed=2, ext=ext)
    ref = oracle.bin_records(*rec[:5], rec[5].astype(bool), n, cams, 16, 16)
    pairs = len(ref["keys"])
    capacity = max(capacity, pairs + 1)
    r = G.renderer(pair_capacity=capacity, flags=_lib.FLAG_DEBUG)
    r.ctx.bin(n, cams, *(torch.from_numpy(a).to(G.DEV) for a in rec))
    r.ctx.check()
    assert np.array_equal(r.ctx.export(_lib.EXPORT_VALUES), ref["values"].astype(np.int32))
    up = lambda a, b: -(-a // b)  # noqa: E731
    passes = 4 * 1024 * up(capacity, 2048)  # four digit tables, a column per 2,048 pairs
    # the depth sort's tables or places, and the histograms of both sorts
    sort = 4 * (1024 * (up(n, 2048) + 2 * 17) + (n if n <= 20480 else 0))
    patches = up(size, 128) ** 2
    rows = 256 * patches * up(n, 256 if n * patches <= 1 << 20 else 1024)
    print("pairs", pairs, "capacity", capacity, "state", state_bytes(r), "passes", passes, "rows", rows, flush=True)
    assert own == (rows > passes)
    assert state_bytes(r) <= max(passes, rows) + sort + 256 * 1024
    small = G.renderer(pair_capacity=64, flags=_lib.FLAG_DEBUG)  # overflow, the rows in room of their own
    small.ctx.bin(n, cams, *(torch.from_numpy(a).to(G.DEV) for a in rec))
    assert not small.ctx.export(_lib.EXPORT_RANGES).any()
