"""Calls on a stream under graph capture: those whose metadata a graph would outlive are refused and leave the
capture and the library as they were; paged_decode_attn_noalloc is captured and replayed."""
import numpy as np
import pytest

from gpu_helpers import note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


def test_calls_under_capture():
    import torch
    B, Hq, Hkv, d, maxp = 4, 8, 2, 64, 8
    pool = kp.Pool(1, B * maxp, Hkv, d)
    bt = torch.arange(B * maxp, dtype=torch.int32, device="cuda").view(B, maxp).contiguous()
    kv = torch.randn(B * 100, Hkv, d, device="cuda").to(torch.bfloat16)
    kp.kv_append(pool, 0, kv, kv, bt, np.zeros(B, np.int32), np.arange(B + 1, dtype=np.int32) * 100)
    lens = np.full(B, 100, np.int32)
    q = torch.randn(B, Hq, d, device="cuda").to(torch.bfloat16)
    out = torch.zeros(B, Hq, d, device="cuda")
    step = np.arange(B + 1, dtype=np.int32)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    q_pf = torch.randn(B, Hq, d, device="cuda").to(torch.bfloat16)
    out_pf = torch.full((B, Hq, d), 3.0, device="cuda")
    s = torch.cuda.Stream()
    tok = torch.arange(64, dtype=torch.int32, device="cuda")
    hashes = torch.zeros(4, dtype=torch.int64, device="cuda")

    def refused():
        yield lambda: kp.kv_append(pool, 0, kv[:B], kv[:B], bt, lens, step, stream=s)
        yield lambda: kp.paged_decode_attn(q, pool, 0, bt, lens, out=out_pf, ws=ws, stream=s)
        yield lambda: kp.prefix_chunk_prefill_attn(q_pf, pool, 0, bt, lens - 1, step, out=out_pf, ws=ws, stream=s)
        yield lambda: kp.kvp_block_hashes(tok, [0, 64], out=hashes, stream=s)

    with torch.cuda.stream(s):  # everything loaded and pinned before the capture
        kp.paged_decode_attn_noalloc(q, pool, 0, bt, lens, out, stream=s)
        kp.paged_decode_attn(q, pool, 0, bt, lens, out=out, ws=ws, stream=s)
    torch.cuda.synchronize()
    note("calls under capture")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for call in refused():
            with pytest.raises(kp.KvpError) as e:
                call()
            assert e.value.code == kp.KVP_EHIP
        kp.paged_decode_attn_noalloc(q, pool, 0, bt, lens, out, stream=s)
    for rep in range(4):
        q.copy_(torch.randn(B, Hq, d, device="cuda"))
        ref = kp.paged_decode_attn(q, pool, 0, bt, lens, out_dtype=torch.float32)
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert bool(torch.all(out_pf == 3.0)) and not bool(hashes.any())
    for call in refused():  # the same calls after the capture, more often than there are blocks
        for _ in range(15):
            call()
    torch.cuda.synchronize()
    assert pool.device_error() == kp.KVP_OK
    pool.close()
