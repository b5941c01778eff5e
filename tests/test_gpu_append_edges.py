"""The append at the edges of its request search and of its workgroups (GPU): batches of 63
to 66 and 300 requests (a scan in one wavefront up to 64, workgroup-wide beyond), requests
without new tokens first, last and between, suffixes that start and end inside, at and around
pages, head counts that leave half of a workgroup idle at head_dim 64. Pools bit for bit
against the oracle, through the append and the combined append-and-plan launch."""
import numpy as np
import pytest

import gpu_helpers as H
from paper_2505_23970_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu_ready():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_23970_amd as gc
    gc.load_library()


def lengths(batch):
    rng = np.random.default_rng(batch)
    P = rng.integers(0, 50, batch)
    n = rng.choice([0, 1, 2, 15, 16, 17, 33], batch)
    n[0] = 0 if batch > 1 else 5
    n[-1] = 0 if batch > 2 else 18
    n[batch // 2] = 40
    return P, n


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("D,Hkv", [(64, 1), (64, 2), (64, 3), (128, 1), (128, 3)])
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 66, 300])
def test_pools_bit_for_bit(batch, D, Hkv, fp8):
    import paper_2505_23970_amd as gc
    P, n = lengths(batch)
    w = W.build(P, n, Hkv, Hkv, D, seed=800 + batch, name=f"append_{batch}_{Hkv}_d{D}")
    print(f"case {w.name} fp8={fp8}: {w.total_new} tokens", flush=True)
    for entry in ("append", "prepare"):
        if fp8:
            run = H.DeviceRunFp8(w, 0.02, 0.015)
            kp_ref, vp_ref = H.oracle_pools_fp8(run)
        else:
            run = H.DeviceRun(w)
            kp_ref, vp_ref = H.oracle_pools(w)
        if entry == "append":
            run.append()
        else:
            ws = gc.alloc_workspace(Hkv, run.k_pool, run.v_pool, run.batch)
            more = dict(k_scale=run.ks, v_scale=run.vs) if fp8 else {}
            gc.prepare(run.k_new, run.v_new, run.k_pool, run.v_pool, run.batch, Hkv, ws, **more)
            assert gc.plan_status(ws) == 0
        kp, vp = run.pools() if fp8 else (H.from_dev_bits(run.k_pool), H.from_dev_bits(run.v_pool))
        assert np.array_equal(kp, kp_ref), f"{entry}: k_pool differs at {np.argwhere(kp != kp_ref)[:5]}"
        assert np.array_equal(vp, vp_ref), f"{entry}: v_pool differs at {np.argwhere(vp != vp_ref)[:5]}"


@pytest.mark.parametrize("D,Hkv,pages", [(128, 1, 512), (128, 1, 513), (64, 3, 256), (64, 3, 257)])
def test_both_sides_of_the_search(D, Hkv, pages):
    """512 workgroups are the last launch whose wavefronts search by themselves."""
    w = W.build([7, 0, 5], [16 * (pages - 3) + 9, 0, 20], Hkv, Hkv, D, seed=900 + pages, name=f"search_{pages}_d{D}")
    assert int(sum(-(-(P + n) // 16) - P // 16 for P, n in zip(w.prefix_lens, w.new_lens) if n)) == pages
    kp_ref, vp_ref = H.oracle_pools(w)
    run = H.DeviceRun(w)
    run.append()
    assert np.array_equal(H.from_dev_bits(run.k_pool), kp_ref)
    assert np.array_equal(H.from_dev_bits(run.v_pool), vp_ref)
