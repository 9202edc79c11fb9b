"""GPU parity of attention at both sides of the rules that pick the workgroups (64 rows of shared blocks, 64, 128 or 256): the
rows of one problem do not depend on the launch they are computed in.  Every case runs alone, repeated in a batch, and three
times in a grouped launch, in the workgroups listed (tests/host/shared_blocks_check.cpp holds the launches to them); the
results are compared bit for bit and with the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # hq, hkv, d, L, l_a, n_p, repeats, rows alone / in the batch / in the group (s: of shared blocks)
    (2, 1, 64, 129, 0, 0, 40),           # s64 / s64 / s64: just over the blocks that always take 64 rows
    (2, 1, 64, 700, 33, 95, 12),         # s64 / s64 / s64: ragged tiles and segments
    (4, 1, 64, 300, 100, 4900, 40),      # s64 / 128 / s64
    (8, 8, 64, 150, 67, 933, 30),        # s64 / s64 / s64: rows 150 to 191 of the last tile missing, no shared K/V
    (4, 2, 128, 129, 7, 0, 3),           # s64 / s64 / s64
    (4, 2, 128, 513, 40, 4000, 20),      # s64 / 256 / s64: a last tile of one row
    (28, 4, 128, 700, 33, 1467, 3),      # 128 / 256 / 256
    (40, 8, 128, 289, 100, 1600, 3),     # s64 / 256 / 256: a last tile of 33 rows
    # the other workgroups of either head_dim
    (8, 4, 64, 77, 20, 50, 40),          # s64 / 64 / s64
    (8, 2, 128, 100, 20, 50, 20),        # s64 / 64 / s64
    (16, 4, 64, 1700, 0, 60, 2),         # s64 / 128 / 128
    (16, 2, 128, 1200, 30, 70, 2),       # s64 / 128 / 128
    (8, 8, 64, 1500, 100, 100, 83),      # s64 / 256 / s64: K and V exceed the caches
]


def bits(rng, shape):
    return wl.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))


def dev(b):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).cuda()


@pytest.mark.parametrize("hq,hkv,d,L,l_a,n_p,repeats", CASES)
def test_rows_do_not_depend_on_the_workgroup(hq, hkv, d, L, l_a, n_p, repeats):
    rng = np.random.default_rng((71, hq, L, n_p))
    host = [bits(rng, (n, h, d)) for n, h in ((L, hq), (l_a, hkv), (l_a, hkv), (n_p, hkv), (n_p, hkv), (L, hkv), (L, hkv))]
    args = [dev(x) for x in host]
    scale = 1.0 / math.sqrt(d)
    print(f"workgroups hq={hq} hkv={hkv} d={d} L={L} l_a={l_a} n_p={n_p} x {repeats}", flush=True)
    out, lse = apbv.apbv_host_attention(*args, scale, return_lse=True)
    def canaries(n):                      # an output of n rows with a row of NaN before and after it
        whole = torch.full((n + 2, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        return whole, whole[1:n + 1]
    whole, many = canaries(repeats * L)
    many, lse_many = apbv.apbv_host_attention(*[x.unsqueeze(0).expand(repeats, *x.shape).contiguous() for x in args], scale, return_lse=True,
                                              out=many.view(repeats, L, hq, d))
    outs = [canaries(L) for _ in range(3)]
    group = apbv.apbv_host_attention_group([tuple(args) + (o,) for _, o in outs], scale, return_lse=True)
    torch.cuda.synchronize()
    ref, lse_r = oracle.host_attention(*host, scale)
    got = wl.bf16_bits_to_f32(out.cpu().view(torch.int16).numpy().view(np.uint16)).astype(np.float64)
    diff = np.abs(got - ref)
    assert diff.max() <= 2e-2 and diff.mean() / np.abs(ref).mean() <= 5e-3
    np.testing.assert_allclose(lse.cpu().numpy().astype(np.float64), lse_r, atol=2e-3, rtol=0)
    for grouped, lse_g in group:
        assert torch.equal(grouped.view(torch.int16), out.view(torch.int16)) and torch.equal(lse_g, lse)
    for w in [whole] + [w for w, _ in outs]:
        assert torch.isnan(w[0]).all() and torch.isnan(w[-1]).all() and not torch.isnan(w[1:-1]).any()
    for b in range(repeats):
        assert torch.equal(many[b].view(torch.int16), out.view(torch.int16)) and torch.equal(lse_many[b], lse)
