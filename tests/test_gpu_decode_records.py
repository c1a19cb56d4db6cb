"""The wave path's chunk records: chunks of one member (held by the record) and of up to 16 (the others looked up),
in calls whose segments hold one chunk and several (records chained past the first ones)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_close, note, to_dev_bits
from oracle import fp8 as F
from paper_2608_11152_amd import kvpattn as kp
from paper_2608_11152_amd import workloads as W

pytestmark = pytest.mark.gpu


# (query heads, KV heads, members of each group, private sequences): 16 / G members fill a chunk's columns.
@pytest.mark.parametrize("Hq,Hkv,groups,singles", [
    (1, 1, [16, 3, 1], 5),        # few chunks, one a segment
    (8, 8, [16, 16, 2], 400),     # more chunks than the call's segments: chains of chunks
    (16, 4, [4, 2, 3], 900),
    (16, 2, [2, 1], 0),
    (16, 1, [1], 3),              # one member a chunk
])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_chunk_records(Hq, Hkv, groups, singles, kv):
    import torch
    d, scale = 64, 0.125
    rng = np.random.default_rng(Hq * 100 + singles)
    shared = [int(rng.integers(1, 4)) for _ in groups]
    gid = sum([[g] * m for g, m in enumerate(groups)], []) + [-1] * singles
    lens = [16 * (shared[g] if g >= 0 else 0) + int(rng.integers(1, 40)) for g in gid]
    pages = [(n + 15) // 16 for n in lens]
    bt = np.zeros((len(lens), max(pages)), np.int32)
    ids, first, used = rng.permutation(sum(pages)).astype(np.int32), {}, 0
    for i, (g, n) in enumerate(zip(gid, pages)):
        s = shared[g] if g >= 0 else 0
        if s and g not in first:
            first[g] = ids[used:used + s]
            used += s
        if s:
            bt[i, :s] = first[g]
        bt[i, s:n] = ids[used:used + n - s]
        used += n - s
    pool = kp.Pool(1, len(ids), Hkv, d, dtype=kp.KVP_FP8_E4M3 if kv == "fp8" else kp.KVP_BF16)
    # every page's content by page id, appended as one long sequence over all the pages
    kvb = W.f32_to_bf16_bits(rng.standard_normal((16 * len(ids), 2, Hkv, d), dtype=np.float32))
    all_pages = torch.arange(len(ids), dtype=torch.int32, device="cuda")[None, :]
    kvd = to_dev_bits(kvb)
    kp.kv_append(pool, 0, kvd[:, 0].contiguous(), kvd[:, 1].contiguous(), all_pages, [0], [0, len(kvb)])
    qb = W.f32_to_bf16_bits(rng.standard_normal((len(lens), Hq, d), dtype=np.float32))
    note(f"chunk records Hq={Hq} Hkv={Hkv} groups={groups} singles={singles} kv={kv}")
    got = kp.paged_decode_attn(to_dev_bits(qb), pool, 0, torch.from_numpy(bt).cuda(), lens, group_prefix=(gid, shared),
                               out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert pool.device_error() == kp.KVP_OK
    content = oracle.widen_bf16(kvb)
    if kv == "fp8":
        content = F.dequantize(F.quantize_bf16(kvb, 1.0), 1.0)
    for i, n in enumerate(lens):
        tok = (bt[i, :pages[i], None] * 16 + np.arange(16)).reshape(-1)[:n]
        ref = oracle.decode_seq(qb[i], content[tok, 0], content[tok, 1], scale)
        assert_close(got[i], ref, f"sequence {i}")
    pool.close()
