"""mixed_step_attn's shared launch against the two calls, bit for bit, and decode and prefill against float64
attention: prefill parts whose own call takes half tiles or whole ones, every GQA ratio, both head sizes and page
types; decode parts of no, few and many wave blocks, wide groups staged through LDS, empty sequences."""
import math

import numpy as np
import pytest

from gpu_helpers import MAX_ABS, MEAN_ABS, note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


# (decode lengths, wide group: members x shared pages, chunks, their history)
PARTS = {
    "one of each": ([1], None, [1], 0),
    "half tiles": ([17, 0, 300, 64], None, [1, 15, 33, 128, 257], 40),
    "half tiles, split": ([500] * 9, None, [3, 70], 1500),
    "whole tiles": ([2000, 3], None, [1, 16, 33, 40] * 8, 1100),
    "empty decodes": ([0, 0, 0], None, [65, 2], 200),
    "wide group": ([], (70, 40), [40, 5], 100),
    "many decodes": ([100 + 7 * i for i in range(300)], None, [20], 600),
}


@pytest.mark.parametrize("parts", PARTS)
@pytest.mark.parametrize("kv,d,G,Hkv", [("bf16", 128, 8, 2), ("bf16", 64, 4, 2), ("fp8", 128, 1, 4), ("fp8", 64, 16, 1),
                                        ("bf16", 128, 2, 1)])
def test_shared_launch(parts, kv, d, G, Hkv):
    import torch
    dec, wide, new, ctx = PARTS[parts]
    gp = None
    shared = 0
    if wide:
        shared = wide[1]
        dec = [shared * 16 + 1 + i % 50 for i in range(wide[0])]
        gp = kp.group_prefix(np.zeros(len(dec), np.int32), [shared])
    lens = list(dec) + [ctx + c for c in new]
    pages = [(n + 15) // 16 for n in lens]
    total = sum(pages)
    g = torch.Generator(device="cuda")
    g.manual_seed(G + d)
    k = torch.randn(total * 16, Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn(total * 16, Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    if kv == "fp8":  # values that E4M3 holds exactly
        k, v = (x.to(torch.float8_e4m3fn).to(torch.bfloat16) for x in (k, v))
    pool = kp.Pool(1, total, Hkv, d, dtype=kp.KVP_FP8_E4M3 if kv == "fp8" else kp.KVP_BF16)
    kp.kv_append(pool, 0, k, v, torch.arange(total, dtype=torch.int32, device="cuda")[None, :], [0], [0, total * 16])
    perm = torch.randperm(total, generator=g, device="cuda").to(torch.int32)
    bt = torch.zeros(len(lens), max(pages), dtype=torch.int32, device="cuda")
    at = 0
    for i, n in enumerate(pages):
        bt[i, :n] = perm[at:at + n]
        at += n
    bt[:len(dec), :shared] = bt[:1, :shared]
    bd, bp = bt[:len(dec)].contiguous(), bt[len(dec):].contiguous()
    cu = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    qd = torch.randn(len(dec), G * Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    qp = torch.randn(sum(new), G * Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    note(f"mixed step, {parts}: {kv} d={d} G={G} Hkv={Hkv}")
    for out_dtype in (torch.float32, torch.bfloat16):
        od, op = kp.mixed_step_attn(pool, 0, qd, bd, dec, qp, bp, [ctx] * len(new), cu, group_prefix=gp,
                                    out_dtype=out_dtype)
        rd = kp.paged_decode_attn(qd, pool, 0, bd, dec, group_prefix=gp, out_dtype=out_dtype)
        rp = kp.prefix_chunk_prefill_attn(qp, pool, 0, bp, [ctx] * len(new), cu, out_dtype=out_dtype)
        assert torch.equal(od, rd) and torch.equal(op, rp)
    assert pool.device_error() == kp.KVP_OK
    some = sorted({0, len(dec) // 2, len(dec) - 1} | {len(dec), len(lens) - 1})
    for i in some:
        ids = bt[i, :pages[i]].long()
        c = 1 if i < len(dec) else new[i - len(dec)]
        q, got = (qd[i:i + 1], od[i:i + 1]) if i < len(dec) else (x[cu[i - len(dec)]:cu[i - len(dec) + 1]] for x in (qp, op))
        if lens[i] == 0:
            assert not bool(got.any())
            continue
        ki, vi = (x.view(total, 16, Hkv, d)[ids].view(-1, Hkv, d)[:lens[i]].double() for x in (k, v))
        hidden = torch.arange(lens[i], device="cuda")[None, :] > (lens[i] - c + torch.arange(c, device="cuda"))[:, None]
        for h in range(G * Hkv):
            s = (q[:, h].double() @ ki[:, h // G].T.contiguous()) / math.sqrt(d)
            ref = torch.softmax(s.masked_fill(hidden, -math.inf), dim=1) @ vi[:, h // G].contiguous()
            err = (got[:, h].double() - ref).abs()
            # rows of few keys are values of up to 4 or 5 themselves: bf16 weights and output round by up to 2^-8 each
            top = MAX_ABS if lens[i] - c >= 300 else 5 * 2.0 ** -7
            assert err.max() <= top and err.mean() <= (MEAN_ABS if lens[i] - c >= 300 else top / 8), (i, h)
    pool.close()
