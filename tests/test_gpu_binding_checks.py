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


def keep_default_stream_busy():
    """An event at the end of a wait on the default stream."""
    import torch
    busy = torch.cuda.Event()
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)   # 0.5 s of the 100 MHz counter, 20 ms or more of the shader clock
    busy.record()
    return busy


@pytest.fixture(scope="module")
def stream(run):
    """A stream that does not share the default stream's hardware queue (few queues serve all
    streams, and work in one queue is done in order)."""
    import torch
    x = torch.zeros(16, device="cuda")
    for _ in range(8):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            x.add_(1)
        busy = keep_default_stream_busy()
        with torch.cuda.stream(s):
            x.add_(1)
        s.synchronize()
        if not busy.query():
            torch.cuda.synchronize()
            return s
    pytest.skip("every stream shares the default stream's queue")


@pytest.mark.parametrize("how", ["current", "given"])
@pytest.mark.parametrize("call", ["kv_append", "run", "prepare", "run_with_append"])
def test_work_runs_on_the_chosen_stream(run, stream, call, how):
    """While the default stream is kept busy, the call's results are there once the chosen stream has
    run: work left on the default stream would still be queued behind the wait."""
    import torch
    import paper_2505_23970_amd as gc
    q, kn, vn, b, scale = run.q, run.k_new, run.v_new, run.batch, run.w.scale
    old = [run.k_pool, run.v_pool]
    new = [t.clone() for t in old]
    gc.kv_append(kn, vn, *new, b)
    kp_ref, vp_ref = H.oracle_pools(run.w)
    assert np.array_equal(H.from_dev_bits(new[0]), kp_ref) and np.array_equal(H.from_dev_bits(new[1]), vp_ref)
    ws = gc.alloc_workspace(q.shape[1], *new, b)
    gc.plan(q.shape[1], *new, b, ws)
    want = gc.run(q, *new, b, scale, ws)
    pools = [t.clone() for t in (new if call == "run" else old)]
    out = torch.full_like(q, float("nan"))
    if call == "prepare":
        ws.zero_()
    s = stream
    kw = {} if how == "current" else {"stream": s}

    def work():
        if call == "kv_append":
            gc.kv_append(kn, vn, *pools, b, **kw)
            return list(zip(pools, new))
        if call == "run_with_append":
            gc.run_with_append(q, kn, vn, *pools, b, scale, ws, out=out, **kw)
            return list(zip(pools + [out], new + [want]))
        if call == "prepare":
            gc.prepare(kn, vn, *pools, b, q.shape[1], ws, **kw)
        gc.run(q, *pools, b, scale, ws, out=out, **kw)
        return list(zip(pools + [out], new + [want]))

    seen = [torch.empty_like(t) for t in pools + [out]]
    busy = keep_default_stream_busy()
    if how == "current":
        with torch.cuda.stream(s):
            pairs = work()
    else:
        pairs = work()
    with torch.cuda.stream(s):
        for t, (got, _) in zip(seen, pairs):
            t.copy_(got)
    s.synchronize()
    assert not busy.query(), "the default stream's wait ended too early to tell the streams apart"
    torch.cuda.synchronize()
    for t, (_, ref) in zip(seen, pairs):
        assert torch.equal(t.view(torch.int16), ref.view(torch.int16))
