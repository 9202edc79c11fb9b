"""GPU parity of the selection that several workgroups share (a few heads of at most 16384 keys), at the edges of its
rule and of its parts, against the oracle: indices and gathered rows bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # hkv, batch, L, l_p, what the keys hold
    (1, 1, 1, 1, "normal"),
    (2, 1, 700, 31, "normal"),           # one part
    (2, 1, 700, 64, "normal"),           # two
    (1, 1, 1024, 1024, "normal"),        # everything selected: the lowest bucket is a candidate
    (2, 1, 16384, 513, "normal"),        # sixteen uneven parts, the largest resident block
    (2, 1, 16385, 513, "normal"),        # one key more: two launches
    (8, 1, 3000, 200, "normal"),         # the most heads that share
    (3, 3, 3000, 200, "normal"),         # one more
    (2, 1, 5000, 2000, "pairs"),         # every score twice: ties inside and across the cut
    (1, 2, 4000, 600, "outlier"),        # one score far above the rest: crowded buckets, the exact path in every part
    (2, 1, 2000, 100, "equal"),          # all scores equal
    (1, 1, 9000, 8192, "normal"),        # the largest sort the LDS holds, no room for more candidates: two launches
    (1, 1, 9000, 8064, "normal"),        # the largest that is shared
    (1, 1, 8192, 8192, "normal"),        # everything of a block that is shared
    (2, 1, 4097, 4097, "pairs"),
    (1, 2, 2, 1, "normal"),              # the smallest
    (2, 2, 16384, 4096, "equal"),        # the exact path with sixteen parts of 256 rows
    (8, 1, 16384, 5000, "outlier"),
]


@pytest.mark.parametrize("hkv,batch,L,l_p,kind", CASES)
def test_shared_selection(hkv, batch, L, l_p, kind):
    rng = np.random.default_rng((61, hkv, L, l_p))
    d, n_q, hq = 64, 3, 2 * hkv

    def bits(shape, scale=1.0):
        return wl.f32_to_bf16_bits((scale * rng.standard_normal(shape)).astype(np.float32))

    q, k, v = bits((batch, n_q, hq, d)), bits((batch, L, hkv, d)), bits((batch, L, hkv, d))
    if kind == "pairs":
        k[:, L // 2:] = k[:, :L - L // 2]
    elif kind == "outlier":
        k = bits((batch, L, hkv, d), 2.0 ** -10)
        k[:, L // 3] = wl.f32_to_bf16_bits(np.float32(64.0) * np.sign(wl.bf16_bits_to_f32(q[:, 0, ::2])))
    elif kind == "equal":
        k[:] = k[:, :1]

    def dev(b):
        return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).cuda()

    print(f"shared selection hkv={hkv} batch={batch} L={L} l_p={l_p} {kind}", flush=True)
    idx, k_c, v_c = (x.cpu() for x in apbv.apbv_compress_kv(dev(q), dev(k), dev(v), l_p))
    for b in range(batch):
        idx_r, kc_r, vc_r, _ = oracle.compress_kv(q[b], k[b], v[b], l_p)
        np.testing.assert_array_equal(idx[b].numpy(), idx_r)
        np.testing.assert_array_equal(k_c[b].view(torch.int16).numpy().view(np.uint16), kc_r)
        np.testing.assert_array_equal(v_c[b].view(torch.int16).numpy().view(np.uint16), vc_r)


@pytest.mark.parametrize("L", [1, 63, 64, 65, 1023, 1024, 1025, 4097, 16384, 16385, 24577])
def test_alike_scores_are_taken_in_index_order(L):
    """The exact path's collection of equal scores, a range of keys a thread or a wave: ranges that end within 64 keys, are
    empty, or hold one tie each; one workgroup a head (2 and 12 heads), shared selection, long blocks."""
    for hkv, kind in ((2, "all"), (2, "few"), (12, "all")):
        rng = np.random.default_rng((89, L, hkv))
        l_p = max(1, L // 3)
        bits = lambda *shape: wl.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
        k, q = np.repeat(bits(1, hkv, 64), L, axis=0), bits(2, hkv, 64)
        if kind == "few":                       # some above the rest, the last key of each run of 64 among them
            better = wl.f32_to_bf16_bits(np.sign(wl.bf16_bits_to_f32(q).sum(0)) * 4)
            k[63::64] = better
            k[-1] = better
        v = rng.integers(0, 1 << 15, (L, hkv, 64), dtype=np.uint16)
        print(f"alike L={L} hkv={hkv} {kind}", flush=True)
        idx, k_c, v_c = (x.cpu() for x in apbv.apbv_compress_kv(dev(q), dev(k), dev(v), l_p))
        idx_r, kc_r, vc_r, _ = oracle.compress_kv(q, k, v, l_p)
        np.testing.assert_array_equal(idx.numpy(), idx_r)
        np.testing.assert_array_equal(k_c.view(torch.int16).numpy().view(np.uint16), kc_r)
        np.testing.assert_array_equal(v_c.view(torch.int16).numpy().view(np.uint16), vc_r)
