"""GPU parity of the scores whose workgroups add up the pooled query themselves (few probe rows), at the edges of its steps
and of its rule (tests/host/compression_rules_check.cpp), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [(d, n_q, group) for d, sizes in ((128, [(1, 1), (5, 3), (2, 8), (17, 1), (16, 4), (13, 5), (20, 8), (23, 7)]),
                                          (64, [(1, 31), (11, 3), (16, 8), (43, 3), (40, 8), (107, 3)])) for n_q, group in sizes]


@pytest.mark.parametrize("d,n_q,group", CASES)
@pytest.mark.parametrize("batch,L", [(1, 700), (2, 1), (1, 129)])
def test_pooled_in_scores(d, n_q, group, batch, L):
    rng = np.random.default_rng((73, d, n_q, group, L))
    hkv, l_p = 2, min(L, 40)
    bits = lambda *s: wl.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    q, k, v = bits(batch, n_q, hkv * group, d), bits(batch, L, hkv, d), bits(batch, L, hkv, d)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
    print(f"pooled scores d={d} n_q={n_q} group={group} batch={batch} L={L}", flush=True)
    wide = dev(np.repeat(q, 2, axis=2))[:, :, ::2]              # a strided view: every second head of a larger block
    idx, _, _, scores = apbv.apbv_compress_kv(wide, dev(k), dev(v), l_p, return_scores=True)
    torch.cuda.synchronize()
    for b in range(batch):
        idx_r, _, _, s_r = oracle.compress_kv(q[b], k[b], v[b], l_p)
        np.testing.assert_array_equal(idx[b].cpu().numpy(), idx_r)
        got = scores[b].cpu().numpy()
        assert np.abs(got - s_r).max() <= 1e-13 * np.abs(s_r).max()      # float64 sums of at most 2^9 exact products, reordered
