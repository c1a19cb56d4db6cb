"""Prefill work lists on both sides of the length up to which the kernels read them from pinned memory: the same
sessions in one call and in short ones (bitwise), back to back without a synchronisation, alone and beside decode
rows; some sessions against float64 attention."""
import math

import numpy as np
import pytest

from gpu_helpers import MAX_ABS, note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


# one KV head and at most one tile a session: the work list has one item per session (rounded up to 8)
@pytest.mark.parametrize("n", [1, 511, 512, 513, 1030])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_work_list_lengths(n, kv):
    import torch
    G, d, step = 4, 64, 90
    rng = np.random.default_rng(n)
    new, ctx = rng.integers(1, 33, n).astype(np.int32), rng.integers(0, 40, n).astype(np.int32)
    pages = (ctx + new + 15) // 16
    total = int(pages.sum())
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k = torch.randn(total * 16, 1, d, generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn(total * 16, 1, d, generator=g, device="cuda").to(torch.bfloat16)
    if kv == "fp8":  # values that E4M3 holds exactly
        k, v = (x.to(torch.float8_e4m3fn).to(torch.bfloat16) for x in (k, v))
    cu = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    q = torch.randn(int(cu[-1]), G, d, generator=g, device="cuda").to(torch.bfloat16)
    first = np.concatenate([[0], np.cumsum(pages)])
    bt_host = np.zeros((n, int(pages.max())), np.int32)
    for i in range(n):
        bt_host[i, :pages[i]] = np.arange(first[i], first[i + 1])
    bt = torch.from_numpy(bt_host).cuda()
    pool = kp.Pool(1, total, 1, d, dtype=kp.KVP_FP8_E4M3 if kv == "fp8" else kp.KVP_BF16)
    kp.kv_append(pool, 0, k, v, torch.arange(total, dtype=torch.int32, device="cuda")[None, :], [0], [0, total * 16])
    note(f"prefill work list of {n} sessions {kv}")
    whole = kp.prefix_chunk_prefill_attn(q, pool, 0, bt, ctx, cu, out_dtype=torch.float32)
    parts = [kp.prefix_chunk_prefill_attn(q[int(cu[i]):int(cu[min(n, i + step)])], pool, 0, bt[i:i + step],
                                          ctx[i:i + step], cu[i:min(n, i + step) + 1] - cu[i],
                                          out_dtype=torch.float32) for i in range(0, n, step)]
    qd = q[:3].contiguous()
    lens = [int(x) for x in (ctx + new)[:3]]
    qd = qd[:len(lens)]
    dec, beside = kp.mixed_step_attn(pool, 0, qd, bt[:len(lens)], lens, q, bt, ctx, cu, out_dtype=torch.float32)
    alone = kp.paged_decode_attn(qd, pool, 0, bt[:len(lens)], lens, out_dtype=torch.float32)
    assert pool.device_error() == kp.KVP_OK
    assert torch.equal(whole, torch.cat(parts)) and torch.equal(whole, beside) and torch.equal(dec, alone)
    for i in sorted({0, n // 2, n - 1}):
        c, h = int(new[i]), int(ctx[i])
        at = int(first[i]) * 16
        ki, vi = (x[at:at + h + c, 0].double() for x in (k, v))
        hidden = torch.arange(h + c, device="cuda")[None, :] > (h + torch.arange(c, device="cuda"))[:, None]
        for j in range(G):
            s = (q[int(cu[i]):int(cu[i + 1]), j].double() @ ki.T.contiguous()) / math.sqrt(d)
            ref = torch.softmax(s.masked_fill(hidden, -math.inf), dim=1) @ vi
            assert (whole[int(cu[i]):int(cu[i + 1]), j].double() - ref).abs().max().item() <= MAX_ABS
    pool.close()
