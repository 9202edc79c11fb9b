"""The calls a sequence-parallel prefill makes of this library, over the range of sizes it makes them at.

Every case is one call of the public entry points as a serving program makes it: inputs resident on the GPU, outputs
and workspace allocated once beforehand, nothing synchronised.  The sizes are those of ``workloads.CONFIGS`` (Qwen2.5-VL
shaped heads, l_a = n/64 and l_p = n/128 of an n-token video) and of the tests and the benchmark.
"""
import math

import torch

import paper_2601_21444_amd as apbv

# (query heads, KV heads, head_dim): the tiny configuration, the 3B and 7B ones, and two of the tests' shapes
HEADS = [(2, 1, 64), (8, 2, 64), (16, 2, 128), (28, 4, 128), (8, 8, 128)]


def listed():
    return [
        # one layer of one virtual host: compression of the local block, then attention over [anchor | passing | local].
        # Smallest configuration (latency and launches), a short video, and the 128K-token video on eight hosts.
        dict(name="layer-tiny", op="layer", batch=1, hq=2, hkv=1, d=64, n_q=8, l_a=64, blocks=3, l_p=32, L=512, keys="normal", lse=False),
        dict(name="layer-8k", op="layer", batch=1, hq=16, hkv=2, d=128, n_q=64, l_a=1024, blocks=3, l_p=512, L=8192, keys="scaled", lse=False),
        dict(name="layer-128k", op="layer", batch=1, hq=16, hkv=2, d=128, n_q=64, l_a=2048, blocks=7, l_p=1024, L=16384, keys="normal", lse=False),
        # two requests whose video does not divide into whole tiles, log-sum-exp wanted for a later merge
        dict(name="attention-ragged", op="attention", batch=2, hq=28, hkv=4, d=128, l_a=333, blocks=3, l_p=77, L=3001, keys="normal", lse=True),
        # a physical host's share of a layer (anchor block, first and last virtual host) in one launch: the largest call
        dict(name="physical-host", op="group", batch=1, hq=28, hkv=4, d=128, l_a=4096, blocks=0, blocks_2=15, l_p=512, L=16384, keys="normal", lse=False),
        # the per-layer compression alone, on keys with the redundancy of video frames
        dict(name="compress-frames", op="compress", batch=1, hq=28, hkv=4, d=128, n_q=64, l_p=2048, L=16384, keys="frames", reducer="sum", scores=False, noalloc=False),
        # many requests' blocks at once: a stream far larger than the caches
        dict(name="compress-many", op="compress", batch=96, hq=16, hkv=2, d=128, n_q=64, l_p=1024, L=16384, keys="normal", reducer="sum", scores=False, noalloc=False),
        # the two other reductions of the score matrix: a physical host's two blocks, and a batch of requests
        dict(name="compress-max", op="compress", batch=2, hq=16, hkv=2, d=128, n_q=64, l_p=1024, L=16384, keys="normal", reducer="max", scores=False, noalloc=False),
        dict(name="compress-mass", op="compress", batch=16, hq=16, hkv=2, d=128, n_q=64, l_p=1024, L=16384, keys="normal", reducer="softmax_sum", scores=False, noalloc=False),
        # the query block over a host's anchor slice and context block (Eq. 5), and one decoding step over the whole video
        dict(name="query-host", op="query", batch=1, hq=16, hkv=2, d=128, n_q=64, l_a=128, n_c=16384, local=False, keys="normal", lse=True),
        dict(name="decode-128k", op="query", batch=1, hq=16, hkv=2, d=128, n_q=1, l_a=2048, n_c=131072, local=True, keys="normal", lse=False),
        # the sixteen virtual hosts' parts of the query block's attention, combined
        dict(name="merge-hosts", op="merge", batch=1, hq=16, hkv=2, d=128, n_q=64, parts=16, lse=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["layer", "layer", "attention", "group", "compress", "compress", "compress", "query", "query", "query", "merge"])
    hq, hkv, d = rng.choice(HEADS)
    keys = rng.choice(["normal", "scaled", "frames"])
    c = dict(op=op, batch=1, hq=hq, hkv=hkv, d=d, keys=keys)
    if op in ("layer", "attention", "group"):
        L = _log_int(rng, 256, 16384)
        c.update(L=L, l_a=rng.randint(0, L // 4), l_p=max(1, L // rng.randint(32, 128)), blocks=rng.randint(0, 15), lse=rng.random() < 0.5)
        if op == "layer":
            c.update(n_q=rng.choice([8, 64]))
        elif op == "attention":
            c.update(batch=rng.randint(1, 4) if L <= 4096 else 1)
        else:
            n = 2 * rng.randint(1, 8) - 1          # virtual hosts h and 2H-1-h: their passing blocks add up to 2H-1
            c.update(blocks=rng.randint(0, n // 2), l_a=max(1, c["l_a"]))
            c.update(blocks_2=n - c["blocks"])
    elif op == "compress":
        reducer = rng.choice(["sum", "sum", "max", "softmax_sum"])
        L = _log_int(rng, 256, 65536)
        batch = _log_int(rng, 1, max(1, min(96, (96 if reducer == "sum" else 16) * 16384 // L)))
        c.update(L=L, l_p=max(1, L // rng.randint(8, 128)), n_q=rng.choice([8, 33, 64]), batch=batch, reducer=reducer, scores=rng.random() < 0.25)
        fits = apbv.apbv_compress_workspace_bytes(batch, hkv, d, L, c["l_p"]) <= apbv.NOALLOC_MAX_WORKSPACE_BYTES
        c.update(noalloc=reducer == "sum" and fits and rng.random() < 0.3)
    elif op == "query":
        c.update(n_q=rng.choice([1, 1, _log_int(rng, 2, 512)]), n_c=_log_int(rng, 1024, 131072), batch=rng.randint(1, 4), local=rng.random() < 0.5, lse=rng.random() < 0.5)
        c.update(l_a=rng.randint(0, c["n_c"] // 8))
    else:
        c.update(n_q=_log_int(rng, 1, 512), parts=rng.randint(2, 64), lse=rng.random() < 0.5)
        del c["keys"]
    return c


# ---- inputs

def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _keys(g, kind, batch, tokens, hkv, d):
    if kind == "frames" and tokens > 0:
        # the tokens of a 4096-token frame share a mean from a random 16-dimensional subspace, plus noise
        n = -(-tokens // 4096)
        basis = torch.randn((batch, n, hkv, d, 16), generator=g, device="cuda")
        z = torch.randn((batch, n, hkv, 1, 16), generator=g, device="cuda")
        mean = ((basis * z).sum(-1) / 4.0).repeat_interleave(4096, dim=1)[:, :tokens]
        return (mean + 0.5 * _normal(g, batch, tokens, hkv, d)).to(torch.bfloat16)
    x = _normal(g, batch, tokens, hkv, d)
    return x * (1.0 / math.sqrt(d)) if kind == "scaled" else x


def _block(g, c, batch, tokens):
    return _keys(g, c["keys"], batch, tokens, c["hkv"], c["d"]), _normal(g, batch, tokens, c["hkv"], c["d"])


def _passing(g, c, blocks, probe):
    """The compressed blocks of `blocks` preceding hosts, as they would be received."""
    hkv, d = c["hkv"], c["d"]
    k, v = [], []
    for _ in range(blocks):
        kb, vb = _block(g, c, c["batch"], c["L"])
        _, kc, vc = apbv.apbv_compress_kv(probe, kb, vb, c["l_p"])
        k.append(kc)
        v.append(vc)
    if not k:
        return (torch.empty((c["batch"], 0, hkv, d), device="cuda", dtype=torch.bfloat16),) * 2
    return torch.cat(k, 1), torch.cat(v, 1)


def _empty(dtype, *shape):
    return torch.empty(shape, device="cuda", dtype=dtype)


def _compress_state(c, probe, k, v):
    b, hkv, d, l_p, L = c["batch"], c["hkv"], c["d"], c["l_p"], c["L"]
    reducer = c.get("reducer", "sum")
    out = dict(idx_out=_empty(torch.int32, b, hkv, l_p), k_c_out=_empty(torch.bfloat16, b, l_p, hkv, d), v_c_out=_empty(torch.bfloat16, b, l_p, hkv, d))
    if c.get("scores"):
        out["scores_out"] = _empty(torch.float64, b, hkv, L)
    kw = dict(out)
    call = apbv.apbv_compress_kv_noalloc
    if not c.get("noalloc"):
        call = apbv.apbv_compress_kv
        nbytes = apbv.apbv_compress_reduced_workspace_bytes(reducer, b, c["hq"], hkv, d, c["n_q"], L, l_p)
        kw.update(workspace=_empty(torch.uint8, max(nbytes, 256)), reducer=reducer, softmax_scale=1.0 / math.sqrt(d))
    # the compressed rows are bit copies: compared as whole 16-bit patterns
    said = {n: t.view(torch.int16) if t.dtype == torch.bfloat16 else t for n, t in out.items()}
    return dict(call=call, args=(probe, k, v, l_p), kw=kw, out=said)


def _attention_out(c, batch, rows):
    o = dict(out=_empty(torch.bfloat16, batch, rows, c["hq"], c["d"]))
    if c["lse"]:
        o.update(lse_out=_empty(torch.float32, batch, c["hq"], rows))
    return o


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    b, hq, hkv, d = c["batch"], c["hq"], c["hkv"], c["d"]
    op, scale = c["op"], 1.0 / math.sqrt(c["d"])
    if op == "merge":
        # parts as the hosts send them: outputs of unit-variance values averaged over many keys, log-sum-exps near log(keys)
        parts = _normal(g, c["parts"], c["n_q"], hq, d) * 0.1
        lse = torch.randn((c["parts"], hq, c["n_q"]), generator=g, device="cuda") + 9.0
        return dict(op=op, calls=[(apbv.apbv_merge_lse, (parts, lse), dict(out=_empty(torch.bfloat16, c["n_q"], hq, d),
                                                                           lse_out=_empty(torch.float32, hq, c["n_q"])))], lse=c["lse"])
    probe = _normal(g, b, c.get("n_q", 64), hq, d)
    if op == "compress":
        s = _compress_state(c, probe, *_block(g, c, b, c["L"]))
        return dict(op=op, calls=[(s["call"], s["args"], s["kw"])], out=s["out"])
    if op == "query":
        ka, va = _block(g, c, b, c["l_a"])
        kc, vc = _block(g, c, b, c["n_c"])
        kl, vl = _block(g, c, b, c["n_q"] if c["local"] else 0)
        n_keys = c["l_a"] + c["n_c"] + kl.shape[1]
        o = _attention_out(c, b, c["n_q"])
        ws = _empty(torch.uint8, max(apbv.apbv_query_attention_workspace_bytes(b, hq, d, c["n_q"], n_keys), 256))
        return dict(op=op, calls=[(apbv.apbv_query_attention, (probe, ka, va, kc, vc, kl, vl, scale), dict(o, workspace=ws))], out=o)
    ka, va = _block(g, c, b, c["l_a"])
    q = _normal(g, b, c["L"], hq, d)
    k, v = _block(g, c, b, c["L"])
    kp, vp = _passing(g, c, c["blocks"], probe)
    if op == "group":
        none = _empty(torch.bfloat16, 0, hkv, d)
        q2 = _normal(g, b, c["L"], hq, d)
        k2, v2 = _block(g, c, b, c["L"])
        kp2, vp2 = _passing(g, c, c["blocks_2"], probe)
        qa = _normal(g, b, c["l_a"], hq, d)
        problems, out = [], []
        for t in ((qa, none, none, none, none, ka, va), (q, ka, va, kp, vp, k, v), (q2, ka, va, kp2, vp2, k2, v2)):
            t = tuple(x[0] if x.dim() == 4 else x for x in t)
            o = {n: x[0] for n, x in _attention_out(c, 1, t[0].shape[0]).items()}
            problems.append(t + tuple(o.values()))
            out.append(o)
        return dict(op=op, calls=[(apbv.apbv_host_attention_group, (problems, scale), {})], out=out)
    o = _attention_out(c, b, c["L"])
    calls, out = [], dict(o)
    if op == "layer":
        s = _compress_state(c, probe, k, v)
        calls.append((s["call"], s["args"], s["kw"]))
        out.update(s["out"])
    calls.append((apbv.apbv_host_attention, (q, ka, va, kp, vp, k, v, scale), dict(o)))
    return dict(op=op, calls=calls, out=out)


def run(state):
    if state["op"] == "merge":
        (call, args, kw), = state["calls"]
        return call(*args, return_lse=True, **kw) if state["lse"] else call(*args, out=kw["out"])
    for call, args, kw in state["calls"]:
        call(*args, **kw)
    return state["out"]


# ---- what a pass cannot do without

def work(case):
    c = case
    b, hq, hkv, d = c["batch"], c["hq"], c["hkv"], c["d"]
    kv_row, q_row = 2 * hkv * d * 2, hq * d * 2          # bytes of a token's K and V, of a token's queries

    def attention(rows, visible, causal):
        pairs = rows * visible + (rows * (rows + 1) // 2 if causal else 0)
        nbytes = 2 * rows * q_row + (visible + (rows if causal else 0)) * kv_row + (4 * hq * rows if c["lse"] else 0)
        return nbytes, 4 * d * pairs * hq

    def compress():
        nbytes = c["n_q"] * q_row + c["L"] * kv_row // 2 + 2 * c["l_p"] * kv_row + 4 * c["l_p"] * hkv
        nbytes += 8 * c["L"] * hkv if c.get("scores") else 0
        # the sum of the logits is one dot product with the pooled query; the other reductions need every logit
        rows = 1 if c.get("reducer", "sum") == "sum" else c["n_q"] * (hq // hkv)
        return nbytes, 2 * rows * c["L"] * d * hkv

    op = c["op"]
    if op == "merge":
        n = c["n_q"] * hq
        return {"bytes": (c["parts"] + 1) * n * d * 2 + (c["parts"] + (1 if c["lse"] else 0)) * n * 4, "flops": 2 * c["parts"] * n * d}
    if op == "compress":
        parts = [compress()]
    elif op == "query":
        parts = [attention(c["n_q"], c["l_a"] + c["n_c"], c["local"])]
    elif op == "group":
        parts = [attention(c["l_a"], 0, True)] + [attention(c["L"], c["l_a"] + n * c["l_p"], True) for n in (c["blocks"], c["blocks_2"])]
    else:
        parts = [attention(c["L"], c["l_a"] + c["blocks"] * c["l_p"], True)] + ([compress()] if op == "layer" else [])
    return {"bytes": b * sum(p[0] for p in parts), "flops": b * sum(p[1] for p in parts)}


def tolerance(case):
    op = case["op"]
    if op == "compress":
        if case["reducer"] == "sum":
            return {"rel": 1e-13, "max": 1e-11}          # float64 sums; the selection they give is exact
        return {"rel": 4e-6, "max": 1e-4, "differ": 2e-3}  # float32 logits: scores closer than that may change places
    if op == "merge":
        return {"rel": 4e-3, "max": 1.6e-2}              # float32 sums, one rounding to bf16 (4 ulp halves)
    # probabilities and outputs rounded to bf16: 2.2e-3 to 2.9e-3 (largest 1.7e-2) from a float64 evaluation
    return {"rel": 1e-2, "max": 7e-2}
