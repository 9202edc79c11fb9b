"""GPU parity of the compression in one launch (many heads of at most 1024 keys), at the edges of its steps and of its rule
(tests/host/compression_rules_check.cpp), against the oracle: indices and gathered rows bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # d, hkv, batch, n_q, group, L, l_p, what the keys hold
    (64, 9, 1, 1, 1, 1, 1, "normal"),
    (128, 3, 3, 2, 3, 2, 1, "normal"),
    (64, 3, 4, 43, 3, 513, 100, "normal"),        # a key more than a round of loads, a probe row more than a step
    (128, 5, 2, 13, 5, 257, 257, "pairs"),        # everything selected, every score twice
    (128, 12, 1, 33, 8, 256, 96, "outlier"),      # the exact path in every part
    (64, 3, 3, 16, 7, 600, 400, "equal"),
    (64, 4, 32, 5, 2, 1023, 33, "normal"),        # one part
    (128, 8, 16, 3, 3, 700, 65, "normal"),        # two
    (128, 16, 16, 2, 2, 1024, 512, "normal"),     # the most keys
    (64, 16, 17, 1024, 1, 1024, 40, "normal"),    # the most probe rows
    (64, 16, 16, 1, 1, 1024, 1024, "normal"),     # one part with the most outputs
    (128, 8, 32, 2, 1, 1024, 1024, "equal"),
    (64, 16, 16, 3, 2, 1024, 1023, "pairs"),
    (64, 16, 16, 1, 2, 1025, 40, "normal"),       # one key more: a launch per step
]


@pytest.mark.parametrize("d,hkv,batch,n_q,group,L,l_p,kind", CASES)
def test_short_blocks(d, hkv, batch, n_q, group, L, l_p, kind):
    rng = np.random.default_rng((97, d, hkv, L, l_p))
    bits = lambda *s: wl.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    q, k, v = bits(batch, n_q, hkv * group, d), bits(batch, L, hkv, d), bits(batch, L, hkv, d)
    if kind == "pairs":
        k[:, L // 2:] = k[:, :L - L // 2]
    elif kind == "outlier":
        k[:, L // 3] = wl.f32_to_bf16_bits(4096 * wl.bf16_bits_to_f32(k[:, L // 3]))
    elif kind == "equal":
        k[:] = k[:, :1]
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
    wide_q, wide_k = dev(np.repeat(q, 2, axis=2))[:, :, ::2], dev(np.repeat(k, 2, axis=1))[:, ::2]     # strided views
    print(f"short blocks d={d} hkv={hkv} batch={batch} n_q={n_q} group={group} L={L} l_p={l_p} {kind}", flush=True)
    idx, k_c, v_c, scores = (x.cpu() for x in apbv.apbv_compress_kv(wide_q, wide_k, dev(v), l_p, return_scores=True))
    for b in sorted({0, batch // 2, batch - 1}):
        idx_r, kc_r, vc_r, s_r = oracle.compress_kv(q[b], k[b], v[b], l_p)
        np.testing.assert_array_equal(idx[b].numpy(), idx_r)
        np.testing.assert_array_equal(k_c[b].view(torch.int16).numpy().view(np.uint16), kc_r)
        np.testing.assert_array_equal(v_c[b].view(torch.int16).numpy().view(np.uint16), vc_r)
        # float64 sums of at most 2^10 exact products and of at most 2^10 rows, reordered
        assert np.abs(scores[b].numpy() - s_r).max() <= 1e-13 * np.abs(s_r).max()
