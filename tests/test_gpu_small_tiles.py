"""Small tiles (decode) at the edges of their pages, tiles, key chunks and merge (GPU).

A wavefront streams 32-key tiles (two 16-key pages) through a two-tile LDS ring and
takes 16 query rows; a split query tile's chunks are merged by one thread group per row
(up to 8 chunks) or by eight. Lengths around every one of those counts, both head
dimensions, both pool types, group sizes that fill the 16 rows or leave some empty;
outputs and log-sum-exps against the fp64 oracle within the bound derived from the
bf16 weights and output."""
import numpy as np
import pytest

import gpu_helpers as H
from paper_2505_23970_amd import workloads as W

pytestmark = pytest.mark.gpu

# keys per request: pages (16), tiles (32), the ring (64), one or two tokens past each
KEYS = [1, 2, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 66, 95, 97, 128, 129, 255, 257]


@pytest.fixture(scope="module", autouse=True)
def gpu_ready():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_23970_amd as gc
    gc.load_library()


def check(w, fp8, split):
    import paper_2505_23970_amd as gc
    print(f"case {w.name} fp8={fp8} split={split}", flush=True)
    if fp8:
        run = H.DeviceRunFp8(w, 0.02, 0.015)
        run.append()
        kp, vp = H.oracle_pools_fp8(run)
        ref, ref_lse = H.oracle_rows_fp8(run, kp, vp)
        vmax = H.e4m3_vmax(vp, run.vs)
    else:
        run = H.DeviceRun(w)
        run.append()
        kp, vp = H.oracle_pools(w)
        ref, ref_lse = H.oracle_rows(w, kp, vp)
        vmax = None
    out, lse = run.attention(kv_split_tiles=split, tiling=gc.TILES_SMALL)
    H.compare_attention(w, out, lse, ref, ref_lse, contract=False, vmax=vmax)


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,n", [(8, 1, 1), (8, 1, 2), (16, 1, 1), (6, 2, 2), (5, 1, 3), (2, 2, 9)])
def test_lengths_around_pages_and_tiles(Hq, Hkv, n, D, fp8):
    new = [min(n, k) for k in KEYS]
    w = W.build([k - m for k, m in zip(KEYS, new)], new, Hq, Hkv, D, seed=500 + n, values="unit",
                name=f"small_{Hq}_{Hkv}_n{n}_d{D}")
    for split in (None, 1, 2):
        check(w, fp8, split)


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("D", [64, 128])
def test_merge_of_few_and_many_chunks(D, fp8):
    """1, 2, 7, 8, 9, 31, 32, 33 and 65 chunks of one tile: one batch of loads and several,
    with and without the eight thread groups per row."""
    chunks = [1, 2, 7, 8, 9, 31, 32, 33, 65]
    for most in (8, 65):
        keys = [32 * c - 5 for c in chunks if c <= most]
        w = W.build([k - 1 for k in keys], [1] * len(keys), 16, 2, D, seed=520 + most, values="peaked",
                    name=f"merge_{most}_d{D}")
        check(w, fp8, 1)


def test_automatic_split_of_one_long_request():
    """One request whose keys are cut into 384-key chunks, and one a token past a chunk."""
    for P in (383, 384, 385, 4099):
        check(W.build([P], [1], 64, 8, 128, seed=530, values="unit", name=f"one_{P}"), False, None)


def test_sharp_rows_keep_a_weight_of_one():
    """The heaviest key's weight is exactly 1 (the offset is the running maximum), so a row
    that one key dominates returns that key's value to fp32 rounding (then bf16)."""
    w = W.build([300], [1], 8, 1, 128, seed=540, name="sharp")
    W.plant_needles(w, [(0, 299)])
    run = H.DeviceRun(w)
    run.append()
    import paper_2505_23970_amd as gc
    out, _ = run.attention(kv_split_tiles=-1, tiling=gc.TILES_SMALL)
    got = H.from_dev_f32(out)
    v = W.bf16_bits_to_f32(w.v_prefix).astype(np.float64)[299, 0]
    # the other keys' weights sum to at most 300 exp2(-scale 256 log2 e + 3) < 1e-8
    assert np.abs(got - v).max() <= 2.0 ** -8 * np.abs(v).max()
