"""The order in which workgroups take their items: on the host for all counts, on the GPU for launches of each kind, most with XCDs
that have no item of the last row (tests/host/arrangement_check.cpp pins their workgroups and orders)."""
import math

import pytest
import torch

import paper_2601_21444_amd as apbv
from test_abi_host import build_and_run_host_check


def test_arrangement(tmp_path):
    res = build_and_run_host_check(tmp_path, "arrangement_check")
    assert res.returncode == 0 and "arrangement ok" in res.stdout, res.stdout + res.stderr


def problem(g, batch, hq, hkv, d, L, n_p):
    q, kp, vp, k, v = (torch.randn((batch, n, h, d), generator=g, device="cuda", dtype=torch.bfloat16)
                       for n, h in ((L, hq), (n_p, hkv), (n_p, hkv), (L, hkv), (L, hkv)))
    none = torch.empty((batch, 0, hkv, d), device="cuda", dtype=torch.bfloat16)
    return q, none, none, kp, vp, k, v


@pytest.mark.gpu
@pytest.mark.parametrize("batch,hq,hkv,d,L,n_p", [
    (3, 8, 2, 128, 1000, 77), (4, 16, 2, 128, 1160, 283), (4, 16, 2, 128, 1536, 33), (3, 28, 4, 128, 1300, 500),   # as many items on each XCD
    (2, 8, 2, 64, 2900, 300),
    (3, 6, 3, 128, 1654, 136), (2, 16, 2, 128, 655, 4),                                # 64-row workgroups, two a unit: folded
    (4, 6, 3, 128, 2674, 572), (2, 6, 3, 128, 2756, 42),                               # 128 rows, two: folded; folded, in turn
    (2, 16, 2, 128, 2111, 130), (2, 16, 2, 128, 2324, 2), (3, 16, 2, 128, 1381, 32),   # more: folded; in turn, folded; threes, folded
    (3, 28, 4, 128, 806, 121), (3, 16, 2, 128, 1610, 559), (3, 28, 4, 128, 794, 1731), # threes; threes, in turn; in turn
    (3, 28, 4, 128, 1084, 36), (3, 16, 2, 128, 2125, 33),                              # in turn, threes; folded, in turn
    (3, 16, 2, 128, 2605, 5), (3, 16, 2, 128, 2728, 47),                               # folded; in turn, folded
    (2, 9, 3, 64, 3273, 1385), (2, 9, 3, 64, 3657, 931), (4, 9, 3, 64, 3110, 110),     # three a unit: folded
    (3, 9, 3, 64, 3704, 1337),                                                         # in turn, folded
    (3, 9, 3, 64, 1357, 48),                                                           # four a unit: in turn
])
def test_every_item_is_computed_once(batch, hq, hkv, d, L, n_p):
    args = problem(torch.Generator(device="cuda").manual_seed(hq * L), batch, hq, hkv, d, L, n_p)
    scale = 1.0 / math.sqrt(d)
    print(f"arrangement {batch} x {hq}/{hkv} x {L} d={d}", flush=True)
    out, lse = apbv.apbv_host_attention(*args, scale, return_lse=True, out=torch.full_like(args[0], float("nan")))
    one = [apbv.apbv_host_attention(*(x[b] for x in args), scale, return_lse=True) for b in range(batch)]
    torch.cuda.synchronize()
    for b in range(batch):
        assert torch.equal(out[b].view(torch.int16), one[b][0].view(torch.int16)) and torch.equal(lse[b], one[b][1])


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,problems", [
    (6, 3, 128, [(1944, 870), (1898, 15)]), (16, 2, 128, [(696, 272), (354, 30)]),                 # 64-row workgroups: folded; folded, in turn
    (6, 3, 128, [(2358, 322), (2549, 1832), (2788, 1320)]),                                        # 128 rows: folded
    (28, 4, 128, [(903, 50), (1299, 1198)]), (16, 2, 128, [(2319, 726), (2047, 1963)]),            # folded; threes, folded
    (28, 4, 128, [(755, 847), (2133, 1218)]), (28, 4, 128, [(1865, 1227), (1224, 1526)]),          # threes; threes, in turn
    (28, 4, 128, [(2161, 47), (1758, 17)]), (28, 4, 128, [(1983, 23), (472, 1812), (2116, 564)]),  # folded; in turn, folded
    (8, 2, 64, [(3515, 33), (1838, 1337), (788, 78)]), (9, 3, 64, [(1907, 58), (2464, 1925), (2994, 1569)]),       # three a unit: folded
    (9, 3, 64, [(3774, 1278), (3413, 307), (3642, 10)]),
    (9, 3, 64, [(1800, 64), (496, 396)]),                                                          # four a unit: in turn
])
def test_every_item_of_a_group_is_computed_once(hq, hkv, d, problems):
    g = torch.Generator(device="cuda").manual_seed(hq * problems[0][0])
    scale = 1.0 / math.sqrt(d)
    parts = [tuple(x[0] for x in problem(g, 1, hq, hkv, d, L, n_p)) for L, n_p in problems]
    outs = [(torch.full_like(p[0], float("nan")), torch.full((hq, p[0].shape[0]), float("nan"), device="cuda")) for p in parts]
    print(f"arrangement {problems} {hq}/{hkv} d={d}", flush=True)
    apbv.apbv_host_attention_group([p + o for p, o in zip(parts, outs)], scale)
    one = [apbv.apbv_host_attention(*p, scale, return_lse=True) for p in parts]
    torch.cuda.synchronize()
    for (out, lse), (out_1, lse_1) in zip(outs, one):
        assert torch.equal(out.view(torch.int16), out_1.view(torch.int16)) and torch.equal(lse, lse_1)
