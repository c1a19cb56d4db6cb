"""The prefill kernel with a workgroup per half tile (short key ranges) and per whole tile, at the edges of a
tile: one row, the last row of the first half, the first of the second, a whole tile and one row more; both
output types, page types and head sizes; and a split history, whose partial states take the same way out.
Against float64 attention on the same values."""
import math

import numpy as np
import pytest

from gpu_helpers import MAX_ABS, MEAN_ABS, note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


# (G, KV heads, history, chunks): rows per tile = 256 = G x positions
SHAPES = {
    "half tiles": (8, 2, 40, [1, 15, 16, 17, 31, 32, 33]),
    "half tiles, one head per group": (1, 1, 0, [1, 127, 128, 129, 255, 256, 257]),
    "half tiles, wide groups": (16, 1, 300, [7, 8, 9, 16, 17]),
    "half tiles, split": (4, 1, 1500, [1, 32, 33, 70]),
    "whole tiles": (8, 8, 660, [1, 15, 16, 17, 31, 32, 33] * 5),
}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kv,d", [("bf16", 128), ("bf16", 64), ("fp8", 128), ("fp8", 64)])
@pytest.mark.parametrize("out_dtype", ["float32", "bfloat16"])
def test_tile_edges(shape, kv, d, out_dtype):
    import torch
    G, Hkv, ctx, new = SHAPES[shape]
    pages = [(ctx + c + 15) // 16 for c in new]
    total = sum(pages)
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * G + d)
    k = torch.randn(total * 16, Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn(total * 16, Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(sum(new), G * Hkv, d, generator=g, device="cuda").to(torch.bfloat16)
    if kv == "fp8":  # values that E4M3 holds exactly
        k, v = (x.to(torch.float8_e4m3fn).to(torch.bfloat16) for x in (k, v))
    pool = kp.Pool(1, total, Hkv, d, dtype=kp.KVP_FP8_E4M3 if kv == "fp8" else kp.KVP_BF16)
    perm = torch.randperm(total, generator=g, device="cuda").to(torch.int32)
    kp.kv_append(pool, 0, k, v, torch.arange(total, dtype=torch.int32, device="cuda")[None, :], [0], [0, total * 16])
    bt = torch.zeros(len(new), max(pages), dtype=torch.int32, device="cuda")
    at = 0
    for i, n in enumerate(pages):
        bt[i, :n] = perm[at:at + n]
        at += n
    cu = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
    note(f"prefill {shape} {kv} d={d} {out_dtype}")
    got = kp.prefix_chunk_prefill_attn(q, pool, 0, bt, [ctx] * len(new), cu, out_dtype=getattr(torch, out_dtype))
    assert pool.device_error() == kp.KVP_OK
    for i, c in enumerate(new):
        ids = bt[i, :pages[i]].long()
        ki, vi = (x.view(total, 16, Hkv, d)[ids].view(-1, Hkv, d)[:ctx + c].double() for x in (k, v))
        qi = q[int(cu[i]):int(cu[i + 1])].double()
        hidden = torch.arange(ctx + c, device="cuda")[None, :] > (ctx + torch.arange(c, device="cuda"))[:, None]
        for h in range(G * Hkv):
            s = (qi[:, h] @ ki[:, h // G].T.contiguous()) / math.sqrt(d)
            ref = torch.softmax(s.masked_fill(hidden, -math.inf), dim=1) @ vi[:, h // G].contiguous()
            err = (got[int(cu[i]):int(cu[i + 1]), h].double() - ref).abs()
            # a row that sees few keys is a value of up to 4 or 5 itself: bf16 weights and output round it by up
            # to 2^-8 relative each
            top = MAX_ABS if ctx >= 300 else 5 * 2.0 ** -7
            assert err.max() <= top and err.mean() <= (MEAN_ABS if ctx >= 300 else top / 8), (c, h, err.max().item())
    pool.close()
