"""128-row tiles over 8-bit pools at head_dim 64 (GPU): launches of more than one round and long enough
run the kernel of three workgroups per compute unit, shorter ones that of two; both against the
oracle's dequantised attention, with tiles and key ranges that end in the middle of a tile."""
import pytest

import gpu_helpers as H
from paper_2505_23970_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix", [(900, 1003, 877, 0, 1300), (40, 3, 77, 0, 130)], ids=["three", "two"])
def test_long_and_short_launches_match_the_oracle(prefix):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_23970_amd as gc
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = [513, 300, 129, 1100, 255]
    w = W.build(list(prefix), n, 32, 32, 64, seed=330, name="three_per_unit")
    kts = [-(-(p + min(q0 + 128, m)) // 64) for p, m in zip(prefix, n) for q0 in range(0, m, 128)]
    long = sum(kts) * 32 >= 13 * 2 * cus
    if len(kts) * 32 <= 2 * cus or long != (prefix[0] == 900):
        pytest.skip(f"not the launch that is meant on {cus} compute units")
    ks, vs = 2.0 ** -6, 0.0213
    run = H.DeviceRunFp8(w, ks, vs)
    run.append()
    kref, vref = H.oracle_pools_fp8(run)
    ws = gc.alloc_workspace(32, run.k_pool, run.v_pool, run.batch)
    gc.plan(32, run.k_pool, run.v_pool, run.batch, ws)
    outs = []
    for _ in range(2):
        out = torch.full(tuple(w.q.shape), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full(tuple(w.q.shape[:2]), float("nan"), dtype=torch.float32, device="cuda")
        gc.run_fp8(run.q, run.k_pool, run.v_pool, run.batch, w.scale, ks, vs, ws, out=out, lse=lse)
        outs.append(out.clone())
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    rows = H.sample_rows(w, seed=60)
    ref_out, ref_lse = H.oracle_rows_fp8(run, kref, vref, rows=rows)
    H.compare_attention(w, out, lse, ref_out, ref_lse, rows=rows, contract=True, vmax=H.e4m3_vmax(vref, vs))
