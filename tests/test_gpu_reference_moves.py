"""GPU parity of attention where the rows' references move in the middle of the pipelined rounds: all rows of a block, one row of
either 16-row block of a wave, the last row; keys whose norms grow along the key axis move them again and again.  Alone (waves
of one 16-row block) and in a batch (waves of two; tests/host/shared_blocks_check.cpp), bit for bit, and with the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu


def dev(b):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16).cuda()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [slice(None), slice(0, 16), slice(31, 32), slice(272, 273), slice(544, 545)])
def test_reference_moves(d, rows):
    rng = np.random.default_rng((31, d, rows.indices(545)[0]))
    hq, hkv, L, n_p, repeats = 2, 1, 545, 1000, 44 if d == 64 else 40
    q, kp, vp, k, v = (rng.standard_normal((n, h, d)).astype(np.float32) for n, h in ((L, hq), (n_p, hkv), (n_p, hkv), (L, hkv), (L, hkv)))
    q[rows] *= 12
    kp *= np.linspace(0.1, 2.0, n_p, dtype=np.float32)[:, None, None]
    none = np.empty((0, hkv, d), dtype=np.float32)
    host = [wl.f32_to_bf16_bits(x) for x in (q, none, none, kp, vp, k, v)]
    args = [dev(x) for x in host]
    scale = 1.0 / math.sqrt(d)
    print(f"reference moves d={d} rows={rows}", flush=True)
    out, lse = apbv.apbv_host_attention(*args, scale, return_lse=True)
    many, lse_many = apbv.apbv_host_attention(*[x.unsqueeze(0).expand(repeats, *x.shape).contiguous() for x in args], scale, return_lse=True)
    torch.cuda.synchronize()
    for b in range(repeats):
        assert torch.equal(many[b].view(torch.int16), out.view(torch.int16)) and torch.equal(lse_many[b], lse)
    ref, lse_r = oracle.host_attention(*host, scale)
    diff = np.abs(wl.bf16_bits_to_f32(out.cpu().view(torch.int16).numpy().view(np.uint16)).astype(np.float64) - ref)
    assert diff.max() <= 2e-2 and diff.mean() / np.abs(ref).mean() <= 5e-3
    # a probability is off by at most half a bf16 step, 2^-8 of itself, and the row sum by no more
    np.testing.assert_allclose(lse.cpu().numpy().astype(np.float64), lse_r, atol=2.0 ** -8, rtol=2e-5)
