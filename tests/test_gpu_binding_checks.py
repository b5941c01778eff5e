"""The binding's tensor checks and stream (GPU): one combined test passes valid tensors, the
single tests still name what is wrong, and work goes to the stream that is current, or given."""
import numpy as np
import pytest

import gpu_helpers as H
from paper_2505_23970_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def run():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return H.DeviceRun(W.build([70, 5], [9, 20], 8, 2, 64, seed=700, name="binding"))


def test_wrong_tensors_are_refused_by_kind(run):
    import torch
    import paper_2505_23970_amd as gc
    k, v, kp, vp, b = run.k_new, run.v_new, run.k_pool, run.v_pool, run.batch
    with pytest.raises(TypeError):
        gc.kv_append(np.zeros(3), v, kp, vp, b)
    with pytest.raises(ValueError):
        gc.kv_append(k.cpu(), v, kp, vp, b)
    with pytest.raises(TypeError):
        gc.kv_append(k.half(), v, kp, vp, b)
    with pytest.raises(ValueError):
        gc.kv_append(k.transpose(1, 2).contiguous().transpose(1, 2), v, kp, vp, b)
    with pytest.raises(ValueError):
        gc.kv_append(k[:-1], v[:-1], kp, vp, b)
    with pytest.raises(ValueError):
        gc.kv_append(k, v, kp, vp.transpose(2, 3).contiguous(), b)
    ws = gc.alloc_workspace(8, kp, vp, b)
    with pytest.raises(ValueError):
        gc.run(run.q[:-1].contiguous(), kp, vp, b, 0.1, ws)
    with pytest.raises(ValueError):
        gc.run(run.q, kp, vp, b, 0.1, ws, out=torch.empty_like(run.q[:-1]))
    with pytest.raises(ValueError):
        gc.run(run.q, kp, vp, b, 0.1, ws, lse=torch.empty(3, 8, device="cuda"))


@pytest.mark.parametrize("how", ["current", "given"])
def test_work_runs_on_the_chosen_stream(run, how):
    """An event recorded on the chosen stream right after the call covers the append."""
    import torch
    import paper_2505_23970_amd as gc
    kp, vp = run.k_pool.clone(), run.v_pool.clone()
    before = kp.view(torch.int16).clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    if how == "current":
        with torch.cuda.stream(s):
            gc.kv_append(run.k_new, run.v_new, kp, vp, run.batch)
    else:
        gc.kv_append(run.k_new, run.v_new, kp, vp, run.batch, stream=s)
    done = torch.cuda.Event()
    done.record(s)
    done.synchronize()
    kp_ref, vp_ref = H.oracle_pools(run.w)
    assert not torch.equal(kp.view(torch.int16), before)
    assert np.array_equal(H.from_dev_bits(kp), kp_ref) and np.array_equal(H.from_dev_bits(vp), vp_ref)
