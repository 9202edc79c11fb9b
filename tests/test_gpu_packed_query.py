"""GPU parity of the key-split launches of apbv_query_attention, whose rows are the queries of all heads of a KV group,
against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu


def dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()


def to_f64(t):
    return wl.bf16_bits_to_f32(t.detach().contiguous().view(torch.int16).cpu().numpy().view(np.uint16)).astype(np.float64)


def rand_bits(rng, shape):
    return wl.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))


def check(out_gpu, ref, what, max_abs=2e-2, mean_rel=5e-3):
    diff = np.abs(out_gpu - ref)
    print(f"{what}: max_abs={diff.max():.3e} mean_rel={diff.mean() / np.abs(ref).mean():.3e}", flush=True)
    assert np.all(np.isfinite(out_gpu))
    assert diff.max() <= max_abs and diff.mean() / np.abs(ref).mean() <= mean_rel


# Rows of a KV group packed together, at the edges of their row tiles (16, 32, 128, 256 rows; 128 and 2048 tokens), of the
# ranges' tiles and with a causal segment whose queries share a tile with others.  Small as they are, most run in a
# workgroup per query head; the same edges in the other kernels follow below.
PACKED_CASES = [
    # hq, hkv, d, batch, n_q, l_a, n_c, local, n_splits
    (8, 1, 128, 1, 2, 0, 64, False, 2),            # 16 rows exactly; a range of one 64-key tile each
    (7, 1, 128, 2, 1, 33, 100, True, 3),           # 7 rows; segments that meet inside a tile
    (9, 1, 64, 1, 2, 5, 1000, True, 2),            # 18 rows: the second block of 16 two rows long
    (16, 1, 64, 1, 2, 0, 449, False, 1000),        # 32 rows exactly; ranges of one tile, a last key alone
    (4, 4, 128, 3, 5, 7, 700, True, 5),            # no group
    (28, 4, 128, 1, 4, 0, 3 * 64 * 7, False, 3),   # 28 rows; 7 64-key tiles a range: odd tile counts per wave
    (11, 1, 128, 1, 3, 17, 300, True, 2),          # 33 rows: the smallest packed workgroup
    (16, 1, 128, 1, 8, 0, 900, True, 4),           # 128 rows exactly
    (3, 1, 64, 2, 43, 1, 500, True, 3),            # 129 rows
    (6, 2, 128, 1, 129, 40, 300, True, 3),         # 129 tokens: 256-row workgroups
    (2, 1, 64, 1, 2048, 0, 200, True, 7),          # the largest packed block, causal
    (2, 1, 64, 1, 2049, 0, 200, True, 7),          # one more: a workgroup per query head
]


@pytest.mark.parametrize("hq,hkv,d,batch,n_q,l_a,n_c,local,n_splits", PACKED_CASES)
def test_packed_query_blocks(hq, hkv, d, batch, n_q, l_a, n_c, local, n_splits):
    rng = np.random.default_rng((77, hq, n_q, n_c))
    n_l = n_q if local else 0
    q = rand_bits(rng, (batch, n_q, hq, d))
    ka, va, kc, vc, kl, vl = (rand_bits(rng, (batch, n, hkv, d)) for n in (l_a, l_a, n_c, n_c, n_l, n_l))
    scale = 1.0 / math.sqrt(d)
    args = [dev(x) for x in (q, ka, va, kc, vc, kl, vl)]
    print(f"packed query block hq={hq} hkv={hkv} d={d} batch={batch} n_q={n_q} keys={l_a}+{n_c}+{n_l} splits={n_splits}", flush=True)
    whole = torch.full((batch, n_q + 2, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda") if batch == 1 else None
    out = whole[:, 1:n_q + 1] if whole is not None else None          # canary rows on both sides
    out, lse = apbv.apbv_query_attention(*args, scale, n_splits=n_splits, return_lse=True, out=out)
    chosen = apbv.apbv_query_attention(*args, scale)
    torch.cuda.synchronize()
    for b in range(batch):
        ref, lse_r = oracle.host_attention(q[b], ka[b], va[b], kc[b], vc[b], kl[b], vl[b], scale)
        check(to_f64(out[b]), ref, f"item {b}, {n_splits} ranges")
        check(to_f64(chosen[b]), ref, f"item {b}, the library's ranges")
        np.testing.assert_allclose(lse[b].cpu().numpy().astype(np.float64), lse_r, atol=2e-3, rtol=0)
    if whole is not None:
        assert torch.isnan(whole[:, 0]).all() and torch.isnan(whole[:, -1]).all()


# The same through the kernel named: batches of two items in turn, large enough that the plan takes it (held to it by
# tests/host/validation_check.cpp).  One range writes the output itself, more go through the merge.
KERNEL_CASES = [
    # kernel, ranges, hq, hkv, d, batch, n_q, l_a, n_c, local, n_splits
    ("wave", 2, 9, 1, 64, 1, 2, 5, 1000, True, 2),              # 18 rows: the second block of 16 two rows long
    ("wave", 1, 16, 1, 64, 1, 2, 0, 449, False, 0),             # 32 rows exactly; a last key alone
    ("wave", 3, 16, 1, 64, 3, 2, 0, 4999, True, 3),             # many tiles a wave, causal
    ("wave", 3, 28, 4, 128, 4, 4, 0, 1344, False, 3),           # 28 rows; 7 64-key tiles a range: odd tile counts per wave
    ("wave", 1, 28, 4, 128, 48, 4, 0, 1344, False, 0),
    ("wave", 8, 1, 1, 64, 24, 1, 0, 1500, False, 0),            # one row
    ("wave", 21, 32, 1, 128, 12, 1, 10, 8990, True, 0),
    ("wave", 157, 2, 1, 64, 1, 1, 33, 39968, False, 0),         # more ranges than a lane of the merge holds; last key alone
    ("packed128", 1, 8, 1, 128, 48, 2, 0, 64, False, 0),        # 16 rows of 128
    ("packed128", 3, 7, 1, 128, 16, 1, 33, 100, True, 3),       # 7 rows; segments that meet inside a tile
    ("packed128", 2, 11, 1, 128, 12, 3, 17, 300, True, 2),      # 33 rows
    ("packed128", 4, 16, 1, 128, 6, 8, 0, 900, True, 4),        # 128 rows exactly
    ("packed128", 6, 4, 4, 128, 3, 5, 7, 700, True, 0),         # no group
    ("packed128", 3, 6, 2, 128, 8, 129, 40, 300, True, 3),      # 387 rows: four tiles
    ("packed128", 3, 8, 1, 64, 8, 300, 40, 300, True, 3),
    ("packed128", 1, 16, 1, 64, 24, 129, 0, 200, True, 0),
    ("packed256", 3, 16, 1, 128, 6, 129, 0, 2000, False, 3),    # 2064 rows: a ninth tile of 16
    ("packed256", 1, 7, 1, 128, 40, 150, 0, 700, False, 0),     # 1050 rows: a fifth tile of 26
    ("packed256", 3, 8, 1, 64, 8, 257, 0, 12000, False, 3),
    ("per_head", 6, 2, 1, 64, 2, 2049, 0, 200, True, 7),        # one query more than the largest packed block
    ("per_head", 2, 8, 2, 128, 1, 2100, 0, 1000, False, 2),     # ... in 256-row workgroups
    ("per_head", 4, 12, 2, 128, 1, 2100, 0, 1540, True, 4),
]


@pytest.mark.parametrize("kernel,ranges,hq,hkv,d,batch,n_q,l_a,n_c,local,n_splits", KERNEL_CASES)
def test_every_kernel_of_the_query_block(kernel, ranges, hq, hkv, d, batch, n_q, l_a, n_c, local, n_splits):
    rng = np.random.default_rng((79, hq, n_q, n_c))
    n_l, distinct = n_q if local else 0, min(batch, 2)
    host = [rand_bits(rng, (distinct, n, h, d)) for n, h in ((n_q, hq), (l_a, hkv), (l_a, hkv), (n_c, hkv), (n_c, hkv), (n_l, hkv), (n_l, hkv))]
    pick = np.arange(batch) % distinct
    scale = 1.0 / math.sqrt(d)
    print(f"{kernel} x {ranges} hq={hq} hkv={hkv} d={d} batch={batch} n_q={n_q} keys={l_a}+{n_c}+{n_l} splits={n_splits}", flush=True)
    whole = torch.full((batch * n_q + 2, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")       # a canary row on both sides
    out, lse = apbv.apbv_query_attention(*[dev(x[pick]) for x in host], scale, n_splits=n_splits, return_lse=True,
                                         out=whole[1:-1].view(batch, n_q, hq, d))
    torch.cuda.synchronize()
    assert torch.isnan(whole[0]).all() and torch.isnan(whole[-1]).all()
    rows = np.unique(np.concatenate([np.arange(min(n_q, 40)), np.arange(max(0, n_q - 40), n_q), rng.integers(0, n_q, 100)]))
    for i in range(distinct):
        ref, lse_r = oracle.host_attention(*[x[i] for x in host], scale, rows=rows)
        items = np.flatnonzero(pick == i)
        check(to_f64(out[items[0]])[rows], ref, f"item {i}")
        np.testing.assert_allclose(lse[items[0]].cpu().numpy().astype(np.float64)[:, rows], lse_r, atol=2e-3, rtol=0)
        for b in items[1:]:
            assert torch.equal(out[b].view(torch.int16), out[items[0]].view(torch.int16)) and torch.equal(lse[b], lse[items[0]])


# Keys whose norms grow or fall along the axis and large logits: the reference maximum moves in most tiles, and waves and
# ranges end with maxima far apart
@pytest.mark.parametrize("gain", [8.0, 40.0])
@pytest.mark.parametrize("order", ["ascending", "descending"])
@pytest.mark.parametrize("hq,hkv,d,batch,n_q,n_c,n_splits", [(16, 1, 64, 1, 1, 5000, 3), (9, 1, 64, 1, 2, 1005, 2), (28, 4, 128, 4, 4, 1344, 3),
                                                             (7, 1, 128, 24, 2, 1500, 0), (16, 1, 128, 6, 8, 900, 4), (8, 1, 64, 8, 300, 340, 3),
                                                             (16, 1, 128, 6, 129, 2000, 3)])
def test_peaked_logits_of_a_query_block(gain, order, hq, hkv, d, batch, n_q, n_c, n_splits):
    rng = np.random.default_rng((80, hq, n_q, n_c))
    ramp = np.linspace(0.05, 1.0, n_c, dtype=np.float32)[:: 1 if order == "ascending" else -1]
    q, v = rand_bits(rng, (n_q, hq, d)), rand_bits(rng, (n_c, hkv, d))
    k = wl.f32_to_bf16_bits(rng.standard_normal((n_c, hkv, d)).astype(np.float32) * ramp[:, None, None] * np.float32(gain))
    e = np.empty((0, hkv, d), dtype=np.uint16)
    scale = 1.0 / math.sqrt(d)
    print(f"peaked query block gain={gain} {order} hq={hq} d={d} batch={batch} n_q={n_q} keys={n_c} splits={n_splits}", flush=True)
    args = [dev(np.stack([x] * batch)) for x in (q, k, v, e, e, e, e)]
    out, lse = apbv.apbv_query_attention(*args, scale, n_splits=n_splits, return_lse=True)
    torch.cuda.synchronize()
    ref, lse_r = oracle.host_attention(q, k, v, e, e, e, e, scale)
    for b in (0, batch - 1):
        got = to_f64(out[b])
        assert np.all(np.isfinite(got))
        diff = np.abs(got - ref)
        # probabilities, partial results and the output rounded to bf16 (2^-9 each) of values up to 5; for the log-sum-exp
        # the rounded probabilities (2^-9) and logits of up to 500 in float32
        assert diff.max() <= 3 * 5 * 2.0 ** -9 and diff.mean() / np.abs(ref).mean() <= 5e-3
        np.testing.assert_allclose(lse[b].cpu().numpy().astype(np.float64), lse_r, rtol=0, atol=5e-3)


def test_query_attention_accepts_the_workspace_of_a_split_per_head():
    """A workspace too small for the library's preferred ranges is used for fewer of them, down to those of a split with
    a tile of rows per query head (two workgroups per compute unit, four 64-key tiles a range); one byte less is refused."""
    rng = np.random.default_rng(78)
    hq, hkv, d, n_q, n_c = 16, 2, 64, 1, 64 * 4 * 20
    q, kc, vc = rand_bits(rng, (1, n_q, hq, d)), rand_bits(rng, (1, n_c, hkv, d)), rand_bits(rng, (1, n_c, hkv, d))
    e = torch.empty((1, 0, hkv, d), dtype=torch.bfloat16, device="cuda")
    args = [dev(q), dev(kc), dev(vc), e, e, e, e]
    part = hq * d * 2 + 256                                            # bf16 output and 64 bytes of lse, each 256-byte aligned
    full = apbv.apbv_query_attention_workspace_bytes(1, hq, d, n_q, n_c)
    least = 20 * part                                                  # ranges of four 64-key tiles
    assert full > least
    ref, _ = oracle.host_attention(q[0], kc[0], vc[0], *(np.empty((0, hkv, d), dtype=np.uint16),) * 4, 0.125)
    for nbytes in (full, least + 3 * part, least):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = apbv.apbv_query_attention(*args, 0.125, workspace=ws)
        torch.cuda.synchronize()
        check(to_f64(out[0]), ref, f"workspace of {nbytes} bytes")
    with pytest.raises(apbv.ApbvError):
        apbv.apbv_query_attention(*args, 0.125, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
