"""The automatic tiling on the CPU (256 compute units assumed without a GPU) around its
lines: the workspace of the automatic plan is that of the tiling the rule names."""
import ctypes

import numpy as np
import pytest

import paper_2505_23970_amd as gc
from test_abi_host import HostBatch, geo


def workspace(lib, g, desc, tiling):
    size = ctypes.c_size_t()
    opt = gc.PlanOptions(0, tiling)
    assert lib.gc_prefix_prefill_workspace_size(ctypes.byref(g), ctypes.byref(desc), ctypes.byref(opt),
                                                ctypes.byref(size)) == 0
    return size.value


@pytest.mark.parametrize("P,n,D,want", [
    # 8 heads per KV head and 8 KV heads: 32 tokens and 8 grid units per wide tile
    ([3999 + 1], [32], 128, gc.TILES_PREFILL),       # 63 key tiles x 8 < 2 x 256
    ([4000 + 64], [32], 128, gc.TILES_WIDE),         # 64 x 8 = 2 x 256
    ([100] * 32, [32] * 32, 128, gc.TILES_WIDE),     # 256 units, 3 key tiles each
    ([60] * 32, [32] * 32, 128, gc.TILES_WIDE),      # 256 units, 2 each: 512
    ([32] * 32, [32] * 32, 128, gc.TILES_PREFILL),   # 256 units, 1 each
    ([900] * 33, [32] * 33, 128, gc.TILES_PREFILL),  # 264 units: between one and two per CU
    ([900] * 64, [32] * 64, 128, gc.TILES_WIDE),     # 512 units
    ([900] * 64, [27] * 64, 128, gc.TILES_PREFILL),  # 84 % full
    ([900] * 64, [32] * 64, 64, gc.TILES_PREFILL),   # d = 64
])
def test_automatic_tiling(P, n, D, want):
    lib = gc.load_library()
    b = HostBatch(np.array(P), np.array(n))
    g = geo(Hq=64, Hkv=8, D=D, maxb=2100)
    sizes = {t: workspace(lib, g, b.desc, t) for t in (gc.TILES_PREFILL, gc.TILES_WIDE)}
    assert sizes[gc.TILES_PREFILL] != sizes[gc.TILES_WIDE]
    assert workspace(lib, g, b.desc, gc.TILES_AUTO) == sizes[want]


def test_a_large_batch_of_short_tiles_fits_the_fixed_scratch():
    """2 million new tokens of 128 query heads on one KV head at d = 64: about 1 million wide
    tiles or 2 million 128-row ones (the automatic choice), without partial rows; the work list
    alone fits the scratch of the call that takes no workspace."""
    lib = gc.load_library()
    b = HostBatch(np.zeros(1660, np.int32), np.full(1660, 1250, np.int32))
    g = geo(Hq=128, Hkv=1, D=64, maxb=2100)
    assert 32 * int(b.n.sum()) < workspace(lib, g, b.desc, gc.TILES_AUTO) <= gc.NOALLOC_SCRATCH_BYTES
