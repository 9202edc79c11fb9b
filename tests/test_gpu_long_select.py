"""GPU parity of the selection of long blocks (24576 keys and more, a few heads: a histogram by several workgroups, then
selection and gather by several), at the edges of its rule, its parts and its buckets, against the oracle: indices and
gathered rows bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # hkv, batch, d, L, l_p, what the keys hold
    (1, 1, 64, 24576, 1, "normal"),          # the shortest, one row
    (1, 1, 64, 24575, 1, "normal"),          # one key less: a workgroup per head
    (2, 1, 64, 24577, 513, "normal"),        # sixteen uneven parts
    (2, 1, 128, 65536, 2000, "normal"),
    (1, 2, 64, 40001, 8192, "normal"),       # the largest selection the LDS sorts
    (1, 1, 64, 40001, 8193, "normal"),       # one more: a workgroup per head
    (1, 1, 64, 17000, 8065, "normal"),       # shorter, where one workgroup's buckets have no room
    (1, 1, 64, 131072, 700, "normal"),       # the longest block of head_dim 64: a full histogram region
    (1, 1, 64, 131073, 700, "normal"),       # one key more
    (1, 1, 128, 140000, 64, "normal"),       # longer with head_dim 128, two parts
    (2, 1, 64, 30000, 33, "normal"),         # one part
    (4, 8, 64, 25000, 200, "normal"),        # the most heads
    (3, 4, 64, 25000, 70, "normal"),         # a row of eight heads and four more
    (3, 11, 64, 25000, 200, "normal"),       # one more
    (2, 1, 64, 30000, 2500, "pairs"),        # every score twice: ties inside and across bins and the cut
    (2, 1, 64, 30000, 900, "ascending"),     # the sample and the parts see different ranges
    (1, 1, 64, 30000, 900, "outlier"),       # one score far above the rest: all others in one coarse bin
    (2, 1, 64, 25000, 300, "equal"),         # no map
    (2, 1, 64, 25000, 300, "two values"),    # one of them taken in part: crowded, the exact path
    (1, 1, 64, 30000, 500, "missed top"),    # the largest scores lie between the sampled ones, beyond the map
    (1, 1, 64, 30000, 8000, "negative"),     # no score above zero
]


@pytest.mark.parametrize("hkv,batch,d,L,l_p,kind", CASES)
def test_long_selection(hkv, batch, d, L, l_p, kind):
    rng = np.random.default_rng((67, hkv, L, l_p))
    n_q, hq = 3, 2 * hkv
    q = rng.standard_normal((batch, n_q, hq, d)).astype(np.float32)
    k = rng.standard_normal((batch, L, hkv, d)).astype(np.float32)
    if kind == "pairs":
        k = np.repeat(k[:, : L // 2], 2, axis=1)
    elif kind == "ascending":
        q = np.abs(q)
        k = (np.abs(k) * np.linspace(0.5, 2.0, L, dtype=np.float32)[None, :, None, None])
    elif kind == "outlier":
        q = np.abs(q)
        k[:, L // 3] = 1e6
    elif kind == "equal":
        k[:] = k[:, :1]
    elif kind == "two values":
        k[:] = np.where((np.arange(L) % 37 == 0)[None, :, None, None], k[:, 1:2], k[:, :1])
    elif kind == "negative":
        q, k = np.abs(q), -np.abs(k)
    elif kind == "missed top":
        q = np.abs(q)
        sampled = (np.arange(256)[:, None] * (L // 256) + np.arange(16)).ravel()
        between = np.setdiff1d(np.arange(60, L, 150), sampled)
        k[:, between] = np.abs(k[:, between]) * 3
    q, k = wl.f32_to_bf16_bits(q), wl.f32_to_bf16_bits(k)
    v = rng.integers(0, 1 << 15, (batch, L, hkv, d), dtype=np.uint16)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
    print(f"long select {hkv} {batch} {d} {L} {l_p} {kind}", flush=True)
    whole = torch.full((batch * l_p + 2, hkv, d), 7, dtype=torch.int16, device="cuda")
    k_c = whole[1:-1].view(torch.bfloat16).view(batch, l_p, hkv, d)
    idx, k_c, v_c = apbv.apbv_compress_kv(dev(q), dev(k), dev(v), l_p, k_c_out=k_c)
    torch.cuda.synchronize()
    bits = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    assert (whole[0] == 7).all() and (whole[-1] == 7).all()
    for b in range(batch):
        idx_r, kc_r, vc_r, _ = oracle.compress_kv(q[b], k[b], v[b], l_p)
        np.testing.assert_array_equal(idx[b].cpu().numpy(), idx_r)
        assert np.array_equal(bits(k_c[b]), kc_r) and np.array_equal(bits(v_c[b]), vc_r)


@pytest.mark.parametrize("reducer", ["max", "softmax_sum"])
def test_long_selection_of_matrix_scores(reducer):
    """The other reductions: the order is the kernel's own reported scores', ties by index."""
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) for s in ((9, 4, 64), (33000, 2, 64), (33000, 2, 64)))
    idx, k_c, v_c, scores = apbv.apbv_compress_kv(q, k, v, 1100, reducer=reducer, softmax_scale=0.125, return_scores=True)
    torch.cuda.synchronize()
    for h in range(2):
        order = np.argsort(-scores[h].cpu().numpy(), kind="stable")[:1100]
        np.testing.assert_array_equal(idx[h].cpu().numpy(), order)
        rows = torch.from_numpy(order.copy()).cuda()
        assert torch.equal(k_c[:, h], k[rows, h]) and torch.equal(v_c[:, h], v[rows, h])


def keys_of_scores(scores):
    """Key rows whose scores under a probe of ones are exactly these float32 values: the sum of three bfloat16 pieces."""
    k = np.zeros(scores.shape + (64,), dtype=np.uint16)
    rest = scores.astype(np.float32)
    for i in range(3):
        k[..., i] = wl.f32_to_bf16_bits(rest)
        rest = rest - wl.bf16_bits_to_f32(k[..., i])
    assert not rest.any()
    return k


CROWDS = [
    # L, l_p, distinct scores on top, how many alike below them, distinct ones below those: the rest lies far below
    (30000, 500, 0, 128, 0),            # as many as a bucket ranks
    (30000, 500, 0, 129, 0),            # one more: its part sorts what it collected
    (30000, 500, 300, 4096, 0),         # a power of two to sort, and a cut among the alike
    (30000, 5000, 700, 4097, 900),      # distinct outputs on both sides
    (40000, 33, 5, 6000, 0),            # one part
    (40000, 8192, 100, 5000, 4000),
    (24576, 8192, 0, 7000, 3000),
    # bins that may not fit beside the others of their part, whose outputs the parts divide: from 8193 - l_p / 16 scores on
    (30000, 8192, 100, 7680, 4000),     # the largest bin one part takes whole
    (30000, 8192, 100, 7681, 4000),     # one more; outputs on both sides of it
    (30000, 8000, 100, 7700, 150),      # it ends inside the last part's share
    (30000, 8192, 511, 7681, 1),        # it begins at the last output of the first share
    (30000, 1000, 999, 20000, 0),       # the last output alone
    (30000, 1024, 128, 9000, 0),        # it begins at a share of its own
    (40000, 40, 3, 9000, 0),            # one part
]


@pytest.mark.parametrize("L,l_p,above,alike,below", CROWDS)
def test_alike_scores_of_a_long_block(L, l_p, above, alike, below):
    rng = np.random.default_rng((71, L, l_p, alike))
    hkv = 2
    scores = np.stack([rng.permutation(np.concatenate([9 + rng.random(above), np.full(alike, 8.5), 8 + 0.2 * rng.random(below),
                                                       rng.standard_normal(L - above - alike - below) - 9])) for _ in range(hkv)]).astype(np.float32)
    k = np.ascontiguousarray(keys_of_scores(scores).transpose(1, 0, 2))
    q = wl.f32_to_bf16_bits(np.ones((1, hkv, 64), dtype=np.float32))
    v = rng.integers(0, 1 << 15, k.shape, dtype=np.uint16)
    dev = lambda x: torch.from_numpy(x.view(np.int16)).view(torch.bfloat16).cuda()
    print(f"alike scores {L} {l_p}: {above} above {alike} above {below}", flush=True)
    idx, k_c, v_c = apbv.apbv_compress_kv(dev(q), dev(k), dev(v), l_p)
    torch.cuda.synchronize()
    idx_r, kc_r, vc_r, s_r = oracle.compress_kv(q, k, v, l_p)
    assert np.array_equal(s_r, scores)
    bits = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    np.testing.assert_array_equal(idx.cpu().numpy(), idx_r)
    assert np.array_equal(bits(k_c), kc_r) and np.array_equal(bits(v_c), vc_r)
