"""decode_merge_kernel's splits of one sequence's output: head rows cut in 1, 2 and 4 (by the number of
partials), at both head sizes and the smallest and largest head counts per KV head."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_close, note, to_dev_bits
from paper_2608_11152_amd import kvpattn as kp
from paper_2608_11152_amd import workloads as W

pytestmark = pytest.mark.gpu


# (query heads, KV heads, head dim, tokens): partials per sequence = 8-page segments, so 128 and 129 partials
# sit on either side of the first cut at d = 128 (16 lanes' rounds of 8), 313 past the second, 1024 past the
# second at d = 64.
@pytest.mark.parametrize("Hq,Hkv,d,n", [(8, 1, 128, 128 * 128), (8, 1, 128, 128 * 128 + 1), (1, 1, 128, 40000),
                                        (4, 4, 64, 40000), (16, 1, 64, 131067)])
@pytest.mark.parametrize("out", ["float32", "bfloat16"])
def test_merge_of_one_long_sequence(Hq, Hkv, d, n, out):
    import torch
    rng = np.random.default_rng(n + d)
    pages = (n + 15) // 16
    bt = rng.permutation(pages).astype(np.int32)[None, :]
    kvb = W.f32_to_bf16_bits(rng.standard_normal((n, 2, Hkv, d), dtype=np.float32))
    qb = W.f32_to_bf16_bits(rng.standard_normal((1, Hq, d), dtype=np.float32))
    pool = kp.Pool(1, pages, Hkv, d)
    btd, kvd = torch.from_numpy(bt).cuda(), to_dev_bits(kvb)
    _, parts, _ = kp.kvp_plan_decode([n], Hq, Hkv)
    note(f"merge of one sequence Hq={Hq} Hkv={Hkv} d={d} n={n}: {parts} partials")
    assert parts >= 128
    kp.kv_append(pool, 0, kvd[:, 0].contiguous(), kvd[:, 1].contiguous(), btd, [0], [0, n])
    got = kp.paged_decode_attn(to_dev_bits(qb), pool, 0, btd, [n], out_dtype=getattr(torch, out))
    assert pool.device_error() == kp.KVP_OK
    ref = oracle.decode_seq(qb[0], oracle.widen_bf16(kvb[:, 0]), oracle.widen_bf16(kvb[:, 1]), 1.0 / np.sqrt(d))
    assert_close(got[0], ref, f"merge of {parts} partials")
    pool.close()
