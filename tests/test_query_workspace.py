"""apbv_query_attention refuses what it refused before its ranges were chosen per KV head: a call whose split per query
head has more than one range needs a workspace that holds those, also where fewer (or no) ranges would now be taken.
Refusals come before any launch, so the C ABI can be called with made-up addresses."""
import pytest

import paper_2601_21444_amd as apbv
from paper_2601_21444_amd.binding import ApbvTensor


def view(tokens, heads, d):
    return ApbvTensor(0x1000 if tokens else None, tokens, heads * d, d, max(tokens, 1) * heads * d)


def ranges_per_head(batch, hq, n_q, n_keys):
    """Two workgroups per compute unit of one query head's 64 (up to 128 queries) or 256 rows, four 64-key tiles a range."""
    tile = 64 if n_q <= 128 else 256
    tiles = -(-n_keys // 64)
    s = min(-(-512 // (-(-n_q // tile) * hq * batch)), max(tiles // 4, 1), tiles, 256)
    return -(-tiles // -(-tiles // s))


@pytest.mark.parametrize("batch,hq,hkv,d,n_q,n_keys", [
    (1, 16, 2, 128, 1, 131072), (4, 28, 4, 128, 512, 131072), (2, 8, 8, 64, 129, 5000), (1, 2, 1, 64, 2048, 9000),
    (1, 2, 1, 64, 2049, 9000), (3, 28, 4, 128, 17, 2000)])
def test_least_workspace(batch, hq, hkv, d, n_q, n_keys):
    rows = batch * n_q * hq
    part = -(-rows * d * 2 // 256) * 256 + -(-rows * 4 // 256) * 256
    least = ranges_per_head(batch, hq, n_q, n_keys) * part
    assert apbv.apbv_query_attention_workspace_bytes(batch, hq, d, n_q, n_keys) >= least > part
    e = view(0, hkv, d)

    def call(ptr, nbytes):
        return apbv.load_library().apbv_query_attention(batch, hq, hkv, d, view(n_q, hq, d), view(n_keys, hkv, d), view(n_keys, hkv, d),
                                                        e, e, e, e, 0.1, 0, 0x2000, None, ptr, nbytes, None)
    assert call(None, 0) == -4 and call(0x100010, 1 << 40) == -4 and call(0x100000, least - 1) == -4
