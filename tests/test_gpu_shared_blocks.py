"""GPU parity of attention where every wave has one 16-row block (few workgroups) with the launches where it has two: every case
runs alone and repeated in a batch large enough for the other kernels (tests/host/shared_blocks_check.cpp holds the rule to both;
blocks of at most 128 rows at head_dim 128 keep waves of one block in the batch too); rows, log-sum-exps and the rows around them
are compared bit for bit, and with the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # hq, hkv, d, L, l_a, n_p, causal, repeats
    (1, 1, 64, 1, 0, 0, True, 600),          # one row, one key: three of four waves without a row
    (2, 1, 128, 17, 5, 0, True, 200),        # the second 16-row half has one row
    (3, 1, 64, 33, 40, 7, True, 200),        # the second block has one row
    (2, 2, 128, 64, 0, 31, True, 150),       # whole blocks, a key tile that straddles the segments
    (1, 1, 128, 65, 3, 64, True, 150),       # a last row tile of one row
    (2, 1, 64, 100, 0, 33, True, 140),
    (1, 1, 128, 128, 10, 100, True, 140),
    (4, 2, 64, 161, 70, 5, True, 70),
    (2, 1, 128, 545, 0, 1000, True, 40),     # pipelined rounds, then the diagonal
    (2, 1, 128, 40, 300, 50, False, 150),    # no causal segment
    (4, 1, 64, 200, 300, 50, False, 60),
]


def bits(rng, shape):
    return wl.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))


def dev(b):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).cuda()


@pytest.mark.parametrize("hq,hkv,d,L,l_a,n_p,causal,repeats", CASES)
def test_shared_blocks(hq, hkv, d, L, l_a, n_p, causal, repeats):
    rng = np.random.default_rng((93, hq, L, n_p))
    n_l = L if causal else 0
    host = [bits(rng, (n, h, d)) for n, h in ((L, hq), (l_a, hkv), (l_a, hkv), (n_p, hkv), (n_p, hkv), (n_l, hkv), (n_l, hkv))]
    host[0][0] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(host[0][0]) * 30)       # a row whose logits move its block's reference
    args = [dev(x) for x in host]
    scale = 1.0 / math.sqrt(d)
    print(f"shared hq={hq} hkv={hkv} d={d} L={L} l_a={l_a} n_p={n_p} causal={causal} x {repeats}", flush=True)
    whole = torch.full((L + 2, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    out, lse = apbv.apbv_host_attention(*args, scale, return_lse=True, out=whole[1:L + 1])
    many, lse_many = apbv.apbv_host_attention(*[x.unsqueeze(0).expand(repeats, *x.shape).contiguous() for x in args], scale, return_lse=True)
    torch.cuda.synchronize()
    assert torch.isnan(whole[0]).all() and torch.isnan(whole[-1]).all() and not torch.isnan(out).any()
    for b in range(repeats):
        assert torch.equal(many[b].view(torch.int16), out.view(torch.int16)) and torch.equal(lse_many[b], lse)
    if causal:
        group = apbv.apbv_host_attention_group([tuple(args)] * 2, scale, return_lse=True)
        torch.cuda.synchronize()
        for grouped, lse_g in group:
            assert torch.equal(grouped.view(torch.int16), out.view(torch.int16)) and torch.equal(lse_g, lse)
        ref, lse_r = oracle.host_attention(*host, scale)
        got = wl.bf16_bits_to_f32(out.cpu().view(torch.int16).numpy().view(np.uint16)).astype(np.float64)
        diff = np.abs(got - ref)
        assert diff.max() <= 2e-2 and diff.mean() / np.abs(ref).mean() <= 5e-3
        np.testing.assert_allclose(lse.cpu().numpy().astype(np.float64), lse_r, atol=2e-3, rtol=2e-5)
