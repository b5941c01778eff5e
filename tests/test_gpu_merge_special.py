"""Infinities, NaN and rows without weight through the merge of split query tiles (GPU): a
split call returns what the unsplit call returns, whatever the number of chunks (its last
batch of loads is padded) and whichever of the merge's two forms runs."""
import numpy as np
import pytest

import gpu_helpers as H
from paper_2505_23970_amd import workloads as W

pytestmark = pytest.mark.gpu

INF, NINF, NAN = 0x7F80, 0xFF80, 0x7FC0   # bf16


def special(D, n, seed):
    """Requests of 100 .. 1300 keys, 16 query heads on 2 KV heads. Key 40 of request 0 holds a value
    of +inf (value row 3) and of -inf (row 5); every key of request 1 scores -inf (its element 0
    is -inf, the queries' 1); key 70 of request 2 is NaN; request 3 is ordinary."""
    P = [130 - n, 400 - n, 257 - n, 1300 - n]
    w = W.build(P, [n] * 4, 16, 2, D, seed=seed, values="unit", name=f"special_d{D}_n{n}")
    w.q[:, :, 0] = 0x3F80
    run = H.DeviceRun(w)
    run.append()
    k, v = H.from_dev_bits(run.k_pool).copy(), H.from_dev_bits(run.v_pool).copy()

    def at(r, key):
        return w.block_tables[r][key // 16], key % 16

    b, s = at(0, 40)
    v[b, :, 3, s], v[b, :, 5, s] = INF, NINF
    for key in range(400):
        b, s = at(1, key)
        k[b, :, s, 0] = NINF
    b, s = at(2, 70)
    k[b, :, s, :] = NAN
    run.k_pool, run.v_pool = H.to_dev_bf16(k), H.to_dev_bf16(v)
    return run


@pytest.mark.parametrize("n,tiling", [(1, "small"), (2, "small"), (20, "prefill"), (20, "wide")])
@pytest.mark.parametrize("D", [64, 128])
def test_split_rows_hold_what_unsplit_rows_hold(D, n, tiling):
    import paper_2505_23970_amd as gc
    til = {"small": gc.TILES_SMALL, "prefill": gc.TILES_PREFILL, "wide": gc.TILES_WIDE}[tiling]
    run = special(D, n, 760)
    want, want_lse = (H.from_dev_f32(x) for x in run.attention(kv_split_tiles=-1, tiling=til))
    # the definition: one infinite value is the row's output there, its other elements are finite;
    # no weight at all gives 0 and -inf, a NaN score gives NaN and -inf
    assert np.isposinf(want[:n, :, 3]).all() and np.isneginf(want[:n, :, 5]).all()
    assert np.isfinite(np.delete(want[:n], [3, 5], axis=2)).all() and np.isfinite(want_lse[:n]).all()
    assert (want[n:2 * n] == 0).all() and np.isneginf(want_lse[n:2 * n]).all()
    assert np.isnan(want[2 * n:3 * n]).all() and np.isneginf(want_lse[2 * n:3 * n]).all()
    assert np.isfinite(want[3 * n:]).all() and np.isfinite(want_lse[3 * n:]).all()
    vmax = float(np.abs(W.bf16_bits_to_f32(np.concatenate([run.w.v_new.ravel(), run.w.v_prefix.ravel()]))).max())
    for split in (1, 2, 3, 5):
        print(f"case {run.w.name} {tiling} split {split}", flush=True)
        got, lse = (H.from_dev_f32(x) for x in run.attention(kv_split_tiles=split, tiling=til))
        fin = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
        assert np.all(np.abs(got[fin] - want[fin]) <= 2 * H.derived_bound(want[fin], vmax))
        assert np.array_equal(np.isneginf(lse), np.isneginf(want_lse)) and not np.isnan(lse).any()
        ok = np.isfinite(want_lse)
        # (both normalisers are sums of bf16 weights within 2^-8 of the exact sum)
        assert np.all(np.abs(lse[ok] - want_lse[ok]) <= 2.0 ** -7 + 2e-5 * np.abs(want_lse[ok]))


def test_automatic_decode_keeps_an_infinite_value():
    """One decode request of 700 keys, which the automatic plan splits at 384."""
    run = H.DeviceRun(W.build([699], [1], 16, 2, 128, seed=761, values="unit", name="inf_auto"))
    run.append()
    v = H.from_dev_bits(run.v_pool).copy()
    v[run.w.block_tables[0][40 // 16], :, 3, 40 % 16] = INF
    run.v_pool = H.to_dev_bf16(v)
    out, lse = (H.from_dev_f32(x) for x in run.attention())
    assert np.isposinf(out[0, :, 3]).all() and np.isfinite(np.delete(out, 3, axis=2)).all()
    assert np.isfinite(lse).all()
