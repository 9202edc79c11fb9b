"""The order in which workgroups take their items: on the host for all counts, on the GPU for launches of each kind."""
import math

import pytest
import torch

import paper_2601_21444_amd as apbv
from test_abi_host import build_and_run_host_check


def test_arrangement(tmp_path):
    res = build_and_run_host_check(tmp_path, "arrangement_check")
    assert res.returncode == 0 and "arrangement ok" in res.stdout, res.stdout + res.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("batch,hq,hkv,d,L,n_p", [
    (3, 8, 2, 128, 1000, 77),      # 64-row workgroups, some units two
    (4, 16, 2, 128, 1160, 283),    # 128 rows: some units three
    (4, 16, 2, 128, 1536, 33),     # 128 rows: every unit three
    (3, 28, 4, 128, 1300, 500),    # more
    (2, 8, 2, 64, 2900, 300),      # head_dim 64: up to four a unit
])
def test_every_item_is_computed_once(batch, hq, hkv, d, L, n_p):
    g = torch.Generator(device="cuda").manual_seed(hq * L)
    q, kp, vp, k, v = (torch.randn((batch, n, h, d), generator=g, device="cuda", dtype=torch.bfloat16)
                       for n, h in ((L, hq), (n_p, hkv), (n_p, hkv), (L, hkv), (L, hkv)))
    none = torch.empty((batch, 0, hkv, d), device="cuda", dtype=torch.bfloat16)
    scale = 1.0 / math.sqrt(d)
    print(f"arrangement {batch} x {hq}/{hkv} x {L} d={d}", flush=True)
    out, lse = apbv.apbv_host_attention(q, none, none, kp, vp, k, v, scale, return_lse=True, out=torch.full_like(q, float("nan")))
    one = [apbv.apbv_host_attention(*(x[b] for x in (q, none, none, kp, vp, k, v)), scale, return_lse=True) for b in range(batch)]
    torch.cuda.synchronize()
    for b in range(batch):
        assert torch.equal(out[b].view(torch.int16), one[b][0].view(torch.int16)) and torch.equal(lse[b], one[b][1])
