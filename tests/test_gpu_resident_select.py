"""GPU parity of the shared selection at the lengths where its kernel holds more scores a thread (1, 2, 4, 8, 12, 16 times
1024 keys), against the oracle: indices and gathered rows bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_21444_amd as apbv
from paper_2601_21444_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 12288, 12289, 16384])
@pytest.mark.parametrize("d,kind", [(64, "pairs"), (128, "last")])
def test_resident_selection(d, kind, L):
    rng = np.random.default_rng((79, d, L))
    hkv, hq, n_q, l_p = 2, 4, 3, 97
    bits = lambda *s: wl.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    q, k, v = bits(n_q, hq, d), bits(L, hkv, d), bits(L, hkv, d)
    if kind == "pairs":                          # every score twice, half a block apart
        k[L - L // 2:] = k[:L // 2]
    else:                                        # the block's last keys are among the best
        k[-3:] = wl.f32_to_bf16_bits(2 * np.sign(wl.bf16_bits_to_f32(q).reshape(n_q, hkv, 2, d).sum((0, 2))))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()
    print(f"resident selection d={d} {kind} L={L}", flush=True)
    idx, k_c, v_c = apbv.apbv_compress_kv(dev(q), dev(k), dev(v), l_p)
    torch.cuda.synchronize()
    idx_r, kc_r, vc_r, _ = oracle.compress_kv(q, k, v, l_p)
    np.testing.assert_array_equal(idx.cpu().numpy(), idx_r)
    assert kind != "last" or set(range(L - 3, L)) <= set(idx_r[0])
    out = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(out(k_c), kc_r) and np.array_equal(out(v_c), vc_r)
