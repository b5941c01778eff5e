"""The calls that a serving program makes on this framework, as cases to measure.

A case is one layer's work for one ragged batch of requests whose context is (partly) in the
paged KV pool: the new tokens' K/V are saved into the pool and their queries attend over the
cached prefix plus themselves; or, for "restore", cached K/V come back from pinned host memory.
Head shapes are those of the Llama-3 models the workloads module names (8B: 32 query and 8 KV
heads; 70B: 64 and 8; head_dim 128), of one GPU's share of the 70B model under tensor
parallelism (8 and 1), and the head_dim 64 shapes of the tests.

How the calls are made ("entry"):
  step       prepare + run: append and plan in one launch, then the attention (a new batch)
  layer      kv_append + run on a plan made before (every layer after the first of a batch)
  fused      run_with_append on a plan made before
  attention  kv_append + prefix_prefill_attention (plan and run) in a kept workspace
  noalloc    kv_append + prefix_prefill_attention_noalloc (programs that cannot allocate)
  restore    kv_restore of the cached prefixes from pinned host memory
and "pools" says whether the pools hold bf16 values or E4M3 codes with one scale per pool.
"""
import math

import numpy as np
import torch

import paper_2505_23970_amd as gc

PAGE = 16
K_SCALE, V_SCALE = 0.0123, 0.0119   # 8-bit pools: about 5.4 standard deviations at code 448

# Lengths of a batch ("traffic"), drawn from the case's own lengths_seed:
#   equal      every request: prefix cached tokens, new new ones
#   turns      cached prefix uniform in prefix/2 .. 3 prefix/2, new tokens uniform in new/4 .. 7 new/4
#   chat       both lognormal around prefix and new (sigma 0.96 and 1.0): multi-turn chats
#   documents  both lognormal around prefix and new (sigma 0.5): questions on cached documents
#   contexts   cached prefix lognormal around prefix (sigma 0.8), every request exactly new new tokens: decode
#   mixed      half the requests misses (new tokens uniform in prefix/16 .. prefix/2), half hits
#              (prefix uniform in prefix/2 .. 2 prefix, new tokens uniform in new/4 .. 7 new/4), shuffled
#   misses     nothing cached; new tokens uniform in new/8 .. 15 new/8
# Prefixes are clipped to 32768 tokens, new tokens to 4096.


def listed():
    return [
        # smallest: one short question on a cached page or two; launches and host work decide
        dict(name="tiny_step", entry="step", pools="bf16", q_heads=4, kv_heads=1, head_dim=64, batch=1,
             traffic="equal", prefix=128, new=32, lse=False, lengths_seed=1),
        # one interactive user's next token: the latency of a single decode step
        dict(name="decode_one_user", entry="layer", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=1,
             traffic="equal", prefix=4099, new=1, lse=False, lengths_seed=2),
        # a decode step of a busy server: one token for each of 32 conversations
        dict(name="decode_batch", entry="layer", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=32,
             traffic="contexts", prefix=4096, new=1, lse=False, lengths_seed=3),
        # the same over 8-bit pools, on a batch that was formed anew
        dict(name="decode_batch_fp8", entry="step", pools="fp8", q_heads=64, kv_heads=8, head_dim=128, batch=32,
             traffic="contexts", prefix=4096, new=1, lse=False, lengths_seed=4),
        # questions of about 20 tokens on cached documents of about 4000
        dict(name="document_questions", entry="step", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=16,
             traffic="documents", prefix=4000, new=20, lse=False, lengths_seed=5),
        # chat turns of the 8B model
        dict(name="chat_8b", entry="step", pools="bf16", q_heads=32, kv_heads=8, head_dim=128, batch=8,
             traffic="turns", prefix=2560, new=288, lse=True, lengths_seed=6),
        # chat turns of the 70B model, append and attention as one call per layer
        dict(name="chat_70b_fused", entry="fused", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=16,
             traffic="chat", prefix=2048, new=200, lse=False, lengths_seed=7),
        # chat turns of the 70B model over 8-bit pools
        dict(name="chat_70b_fp8", entry="step", pools="fp8", q_heads=64, kv_heads=8, head_dim=128, batch=16,
             traffic="chat", prefix=2048, new=200, lse=False, lengths_seed=8),
        # misses only, head_dim 64: plain causal prefill of a small model
        dict(name="misses_d64", entry="attention", pools="bf16", q_heads=32, kv_heads=8, head_dim=64, batch=16,
             traffic="misses", prefix=0, new=800, lse=True, lengths_seed=9),
        # 128 new tokens on a 32k-token cached context
        dict(name="long_reuse", entry="layer", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=4,
             traffic="equal", prefix=32768, new=128, lse=False, lengths_seed=10),
        # hits' contexts coming back from the cache's host tier
        dict(name="restore_host", entry="restore", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=4,
             traffic="chat", prefix=2048, new=200, lse=False, lengths_seed=11),
        # largest: a mixed batch of 16 misses and 16 hits on long contexts
        dict(name="mixed_70b", entry="step", pools="bf16", q_heads=64, kv_heads=8, head_dim=128, batch=32,
             traffic="mixed", prefix=8192, new=144, lse=False, lengths_seed=12),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tiny", "decode", "decode", "questions", "turns", "turns", "long", "misses", "restore", "mixed"])
    heads = rng.choice([(64, 8, 128), (64, 8, 128), (32, 8, 128), (8, 1, 128), (32, 8, 64), (16, 2, 128)])
    c = dict(pools=rng.choice(["bf16", "bf16", "fp8"]), entry=rng.choice(["step", "layer", "fused", "attention"]),
             lse=rng.random() < 0.3, lengths_seed=rng.randrange(1 << 30))
    if kind == "tiny":
        heads = rng.choice([(4, 1, 64), (8, 1, 128), (4, 4, 64)])
        c.update(batch=rng.randint(1, 4), traffic=rng.choice(["equal", "turns"]), prefix=_log_uniform(rng, 16, 512),
                 new=_log_uniform(rng, 4, 64))
    elif kind == "decode":
        c.update(batch=_log_uniform(rng, 1, 64), traffic="contexts", prefix=_log_uniform(rng, 512, 8192),
                 new=1 if rng.random() < 0.8 else 2, entry=rng.choice(["step", "layer", "attention", "noalloc"]))
        if c["entry"] == "noalloc":
            c["pools"] = "bf16"
    elif kind == "questions":
        c.update(batch=_log_uniform(rng, 1, 32), traffic="documents", prefix=_log_uniform(rng, 1000, 8000),
                 new=_log_uniform(rng, 6, 60))
    elif kind == "turns":
        c.update(batch=_log_uniform(rng, 1, 24), traffic=rng.choice(["turns", "chat"]),
                 prefix=_log_uniform(rng, 500, 5000), new=_log_uniform(rng, 60, 600))
    elif kind == "long":
        c.update(batch=rng.randint(1, 4), traffic="equal", prefix=_log_uniform(rng, 16000, 32768),
                 new=_log_uniform(rng, 16, 256))
    elif kind == "misses":
        c.update(batch=_log_uniform(rng, 1, 16), traffic="misses", prefix=0, new=_log_uniform(rng, 100, 2000))
    elif kind == "restore":
        c.update(batch=rng.randint(1, 6), traffic="chat", prefix=_log_uniform(rng, 256, 3000), new=200,
                 entry="restore", pools="bf16")
    else:
        c.update(batch=2 * rng.randint(2, 16), traffic="mixed", prefix=_log_uniform(rng, 2048, 8192),
                 new=_log_uniform(rng, 64, 200))
    c.update(q_heads=heads[0], kv_heads=heads[1], head_dim=heads[2])
    if c["entry"] in ("fused", "restore", "noalloc"):
        c["pools"] = "bf16"
    largest = work(listed()[-1])
    while c["batch"] > 1 and any(work(c)[k] > largest[k] for k in largest):
        c["batch"] //= 2
    return c


def lengths(case):
    """(cached tokens, new tokens) of every request, int64 arrays."""
    rng = np.random.default_rng(case["lengths_seed"])
    B, prefix, new = case["batch"], case["prefix"], case["new"]
    uniform = lambda lo, hi, size: rng.integers(max(1, int(lo)), max(1, int(hi)), size=size, endpoint=True)  # noqa: E731
    lognormal = lambda median, sigma: np.rint(median * np.exp(sigma * rng.standard_normal(B)))  # noqa: E731
    kind = case["traffic"]
    if kind == "equal":
        P, n = np.full(B, prefix), np.full(B, new)
    elif kind == "turns":
        P, n = uniform(prefix / 2, 1.5 * prefix, B), uniform(new / 4, 1.75 * new, B)
    elif kind == "chat":
        P, n = np.clip(lognormal(prefix, 0.96), 1, 4 * prefix), np.clip(lognormal(new, 1.0), 1, 5 * new)
    elif kind == "documents":
        P, n = np.clip(lognormal(prefix, 0.5), 1, 4 * prefix), np.clip(lognormal(new, 0.5), 4, 64)
    elif kind == "contexts":
        P, n = np.clip(lognormal(prefix, 0.8), 256, None), np.full(B, new)
    elif kind == "mixed":
        h = B // 2
        P = np.concatenate([np.zeros(h), uniform(prefix / 2, 2 * prefix, B - h)])
        n = np.concatenate([uniform(prefix / 16, prefix / 2, h), uniform(new / 4, 1.75 * new, B - h)])
        order = rng.permutation(B)
        P, n = P[order], n[order]
    elif kind == "misses":
        P, n = np.zeros(B), uniform(new / 8, 1.875 * new, B)
    else:
        raise ValueError(kind)
    return np.minimum(P, 32768).astype(np.int64), np.clip(n, 1, 4096).astype(np.int64)


def work(case):
    P, n = lengths(case)
    Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
    elem = 1 if case["pools"] == "fp8" else 2
    row = 2 * Hkv * D                      # elements of one token's K and V
    if case["entry"] == "restore":
        return {"bytes": int(2 * 2 * row * P.sum()), "flops": 0}
    T = int(n.sum())
    pairs = float(np.sum(n * P + n * (n + 1) / 2))
    moved = elem * row * int(P.sum()) + (2 + elem) * row * T + 2 * 2 * Hq * D * T + (4 * Hq * T if case["lse"] else 0)
    return {"bytes": int(moved), "flops": 4.0 * D * Hq * pairs}


# ------------------------------------------------------------------------------- inputs

def _codes(x, scale):
    """E4M3 codes nearest to x / scale (the append's rounding: times fl32(1 / scale), saturated at 448)."""
    inv = np.float32(1) / np.float32(scale)
    return (x.float() * float(inv)).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)


def _inputs(case, seed):
    """Queries and keys of unit variance, the query heads at temperatures from 0.5 to 3 (from nearly
    uniform to sharp attention); the pool is full (other requests' and stale tokens around this batch's)
    and the batch's pages lie in it in random order."""
    P, n = lengths(case)
    Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
    rng = np.random.default_rng(seed)
    pages = -(-(P + n) // PAGE)
    used = int(pages.sum())
    blocks = used + used // 4 + 1
    order = rng.permutation(blocks).astype(np.int32)
    tables = np.zeros((case["batch"], int(pages.max()) + 1), np.int32)
    at = 0
    for r, k in enumerate(pages):
        tables[r, :k] = order[at:at + k]
        at += int(k)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    normal = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    T = int(n.sum())
    x = dict(P=P, n=n, tables=tables, scale=1.0 / math.sqrt(D))
    if case["entry"] == "restore":
        S = int(P.sum())
        x.update(k_host=normal(S, Hkv, D).cpu().pin_memory(), v_host=normal(S, Hkv, D).cpu().pin_memory())
    else:
        heat = 0.5 * 6.0 ** (torch.arange(Hq, device="cuda") / max(1, Hq - 1))
        x.update(q=(normal(T, Hq, D) * heat.to(torch.bfloat16)[None, :, None]).contiguous(),
                 k_new=normal(T, Hkv, D), v_new=normal(T, Hkv, D))
    k_pool, v_pool = normal(blocks, Hkv, PAGE, D), normal(blocks, Hkv, D, PAGE)
    if case["pools"] == "fp8":
        k_pool, v_pool = _codes(k_pool, K_SCALE), _codes(v_pool, V_SCALE)
    x.update(k_pool=k_pool, v_pool=v_pool)
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["batch"] = gc.PagedBatch(s["P"], s["n"], s["tables"], device="cuda")
    if case["entry"] == "restore":
        return s
    Hq = case["q_heads"]
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty(s["q"].shape[:2], dtype=torch.float32, device="cuda") if case["lse"] else None
    if case["entry"] != "noalloc":
        s["workspace"] = gc.alloc_workspace(Hq, s["k_pool"], s["v_pool"], s["batch"])
    if case["entry"] in ("layer", "fused"):
        gc.plan(Hq, s["k_pool"], s["v_pool"], s["batch"], s["workspace"])
    return s


def run(s):
    entry, fp8 = s["case"]["entry"], s["case"]["pools"] == "fp8"
    batch, kp, vp = s["batch"], s["k_pool"], s["v_pool"]
    if entry == "restore":
        gc.kv_restore(s["k_host"], s["v_host"], kp, vp, batch)
        return {"k_pool": kp, "v_pool": vp}
    q, kn, vn, scale, out, lse = s["q"], s["k_new"], s["v_new"], s["scale"], s["out"], s["lse"]
    if entry == "fused":
        gc.run_with_append(q, kn, vn, kp, vp, batch, scale, s["workspace"], out=out, lse=lse)
    else:
        if entry == "step":
            more = dict(k_scale=K_SCALE, v_scale=V_SCALE) if fp8 else {}
            gc.prepare(kn, vn, kp, vp, batch, q.shape[1], s["workspace"], **more)
        elif fp8:
            gc.kv_append_fp8(kn, vn, kp, vp, batch, K_SCALE, V_SCALE)
        else:
            gc.kv_append(kn, vn, kp, vp, batch)
        if entry == "attention" and fp8:
            gc.prefix_prefill_attention_fp8(q, kp, vp, batch, scale, K_SCALE, V_SCALE, s["workspace"], out=out, lse=lse)
        elif entry == "attention":
            gc.prefix_prefill_attention(q, kp, vp, batch, scale, s["workspace"], out=out, lse=lse)
        elif entry == "noalloc":
            gc.prefix_prefill_attention_noalloc(q, kp, vp, batch, scale, out=out, lse=lse)
        elif fp8:
            gc.run_fp8(q, kp, vp, batch, scale, K_SCALE, V_SCALE, s["workspace"], out=out, lse=lse)
        else:
            gc.run(q, kp, vp, batch, scale, s["workspace"], out=out, lse=lse)
    got = {"out": out, "k_pool": kp, "v_pool": vp}
    if lse is not None:
        got["lse"] = lse
    return got


# ------------------------------------------------------------------------------- what is right

def tolerance(case):
    """Restored bytes and 8-bit codes are exact. The attention's outputs are bf16 (each rounded by up to
    2^-9 of itself) of sums whose weights are rounded to bf16 too; another correct order of the sums and
    another exponent offset move the result by about one such rounding. Measured between key splits and
    tilings of the same call: up to 2.9e-3 (2-norm) and 5e-2 (largest element); about four times that, and
    three times, are allowed."""
    if case["entry"] == "restore":
        return "exact"
    return {"rel": 0.012, "max": 0.15, "differ": 0.0}


def exact(case, seed):
    """The attention in float64 over the values that the pools hold after the append (8-bit pools: code
    value times scale), and the pools' new contents as they are (copied or quantised, not computed in 64 bits)."""
    x = _inputs(case, seed)
    P, n, tables = x["P"], x["n"], x["tables"]
    Hq, Hkv, D = case["q_heads"], case["kv_heads"], case["head_dim"]
    g = Hq // Hkv
    kp, vp = x["k_pool"], x["v_pool"]
    fp8 = case["pools"] == "fp8"
    if case["entry"] == "restore":
        new_k, new_v, first, count = x["k_host"].cuda(), x["v_host"].cuda(), np.zeros_like(P), P
    else:
        new_k, new_v, first, count = x["k_new"], x["v_new"], P, n
        if fp8:
            new_k, new_v = _codes(new_k, K_SCALE), _codes(new_v, V_SCALE)
    at = 0
    for r in range(case["batch"]):
        pos = np.arange(first[r], first[r] + count[r])
        block = torch.from_numpy(tables[r][pos // PAGE].astype(np.int64)).cuda()
        slot = torch.from_numpy(pos % PAGE).cuda()
        kp[block, :, slot, :] = new_k[at:at + len(pos)]
        vp[block, :, :, slot] = new_v[at:at + len(pos)]
        at += len(pos)
    if case["entry"] == "restore":
        return {"k_pool": kp, "v_pool": vp}
    value = lambda codes, scale: (codes.view(torch.float8_e4m3fn).double() * float(np.float32(scale))  # noqa: E731
                                  if fp8 else codes.double())
    T = int(n.sum())
    out = torch.empty((T, Hq, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((T, Hq), dtype=torch.float64, device="cuda")
    cu = 0
    for r in range(case["batch"]):
        L, m = int(P[r] + n[r]), int(n[r])
        block = torch.from_numpy(tables[r][:-(-L // PAGE)].astype(np.int64)).cuda()
        for h in range(Hkv):
            k = value(kp[block, h].reshape(-1, D)[:L].contiguous(), K_SCALE)
            v = value(vp[block, h].transpose(1, 2).reshape(-1, D)[:L].contiguous(), V_SCALE)
            kt = k.t().contiguous()
            step = max(1, (1 << 26) // (L * g))
            for i in range(0, m, step):
                j = min(m, i + step)
                q = x["q"][cu + i:cu + j, h * g:(h + 1) * g].double().reshape(-1, D)
                s = torch.mm(q, kt) * float(np.float32(x["scale"]))
                last = torch.arange(int(P[r]) + i, int(P[r]) + j, device="cuda").repeat_interleave(g)
                s.masked_fill_(torch.arange(L, device="cuda")[None, :] > last[:, None], -math.inf)
                total = torch.logsumexp(s, dim=1)
                s.sub_(total[:, None]).exp_()
                out[cu + i:cu + j, h * g:(h + 1) * g] = torch.mm(s, v).reshape(j - i, g, D)
                lse[cu + i:cu + j, h * g:(h + 1) * g] = total.reshape(j - i, g)
        cu += m
    got = {"out": out, "k_pool": None, "v_pool": None}
    if case["lse"]:
        got["lse"] = lse
    return got
