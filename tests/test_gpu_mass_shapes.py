"""GPU parity of the attention-mass reduction at the edges of the kernel that keeps the probe rows in LDS, against the
fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # hq, hkv, d, n_q, batch, L: rows per KV head n_q * hq / hkv; 192 to 512 rows of 128, 384 to 1024 of 64 are resident
    (1, 1, 128, 160, 1, 300),       # one tile of rows too few
    (1, 1, 128, 161, 1, 63),        # 192 rows with padding; less than one block of keys
    (1, 1, 128, 192, 1, 64),        # exactly; one block
    (2, 1, 128, 256, 1, 65),        # 512 rows; a second block of one key
    (1, 1, 128, 513, 1, 200),       # too many
    (3, 1, 128, 87, 2, 1000),       # 261 rows (an odd number of tiles), two items
    (2, 2, 64, 384, 1, 257),        # rows of 64
    (1, 1, 64, 1024, 1, 129),
    (8, 2, 128, 64, 9, 16500),      # blocks that leave the last round of workgroups ragged
    # (192 rows and few keys are streamed all the same, plan_mass; the same edges where the rows are resident)
    (2, 1, 128, 256, 1, 63),        # 512 rows, less than one block of keys
    (2, 1, 128, 256, 1, 64),        # one block
    (1, 1, 128, 161, 1, 70001),     # 192 rows with padding, 1094 blocks
    (1, 1, 128, 192, 1, 70001),     # 192 rows
    (1, 1, 64, 384, 1, 70001),      # 384 rows of 64
    (16, 2, 128, 64, 17, 9000),     # three blocks a wave, a last round of workgroups that is ragged
    (4, 4, 64, 576, 25, 1280),      # and rows that would fit streamed: rounds that do not fill
]


def bits(rng, shape):
    return wl.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))


def dev(b):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).cuda()


@pytest.mark.parametrize("hq,hkv,d,n_q,batch,L", CASES)
def test_mass_at_the_edges_of_the_resident_probe(hq, hkv, d, n_q, batch, L):
    rng = np.random.default_rng((91, n_q, L))
    # (a batch repeats two items: the oracle is the slow side)
    q, k = (bits(rng, (min(batch, 2), n, h, d)) for n, h in ((n_q, hq), (L, hkv)))
    pick = np.arange(batch) % q.shape[0]
    scale, l_p = 1.0 / math.sqrt(d), min(L, 17)
    wide = torch.zeros((batch, L, hkv, d + 8), dtype=torch.bfloat16, device="cuda")       # padded rows: a strided view
    wide[..., :d] = dev(k[pick])
    print(f"mass hq={hq} hkv={hkv} d={d} n_q={n_q} batch={batch} L={L}", flush=True)
    _, _, _, s = apbv.apbv_compress_kv(dev(q[pick]), wide[..., :d], wide[..., :d], l_p, reducer="softmax_sum", softmax_scale=scale, return_scores=True)
    torch.cuda.synchronize()
    s = s.cpu().numpy()
    for i in range(q.shape[0]):
        ref = oracle.importance_scores_softmax_sum(q[i], k[i], scale)
        for b in np.flatnonzero(pick == i):
            # float32 logits, exponentials and sums: the bound of test_gpu_reducers.py, relative to the largest score
            assert np.abs(s[b] - ref).max() <= 5e-6 * np.abs(ref).max()
