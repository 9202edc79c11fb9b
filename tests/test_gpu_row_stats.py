"""GPU parity of the attention-mass scores over the numbers of key chunks and rows at which the merge of the row statistics
takes another step (16 waves of one or eight chunks, 64 rows a workgroup), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q,L", [(1, 1), (16, 256), (17, 257), (32, 4096), (33, 4097), (5, 32768), (3, 33000)])
def test_row_statistics(n_q, L):
    rng = np.random.default_rng((83, n_q, L))
    hq, hkv, d, scale = 4, 2, 64, 0.125
    bits = lambda *s: wl.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    q, k = bits(n_q, hq, d), bits(L, hkv, d)
    q[0] = wl.f32_to_bf16_bits(4 * wl.bf16_bits_to_f32(q[0]))       # a row whose chunks' maxima lie far apart
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
    print(f"row statistics n_q={n_q} L={L}", flush=True)
    _, _, _, scores = apbv.apbv_compress_kv(dev(q), dev(k), dev(k), 1, reducer="softmax_sum", softmax_scale=scale, return_scores=True)
    torch.cuda.synchronize()
    ref = oracle.importance_scores_softmax_sum(q, k, scale)
    got = scores.cpu().numpy()
    # float32 logits and sums: an exponent of up to 2^5 in the log2 domain carries 2^-19, a score's sum of R such terms less
    assert np.abs(got - ref).max() <= 4e-6 * np.abs(ref).max()
    np.testing.assert_allclose(got.sum(1), np.full(hkv, n_q * hq // hkv), rtol=4e-6)      # every row's mass is one
