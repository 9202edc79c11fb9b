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


# Rows of a KV group packed together, at the edges of their row tiles
# (16, 32, 128, 256 rows; 128 and 2048 tokens), of the ranges' tiles (1 to 4 tiles a wave, odd counts, a last key alone)
# and with a causal segment whose queries share a tile with others
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
