"""Pinned metadata blocks turned over while the GPU is behind: a block is written again only after the work
that read it, on one stream and on more streams than blocks stay open for."""
import numpy as np
import pytest

from gpu_helpers import note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_streams,calls", [(1, 80), (6, 60)])
def test_metadata_blocks_under_pending_work(n_streams, calls):
    """Each call's page runs take about 190 KB of a 1 MB block: the calls go through every block and wait for
    the first.  Call c writes every sequence's token at position c of its stream's pages; a block handed out
    too early would give an earlier call a later one's positions."""
    import torch
    B, maxp, Hkv, d = 8000, (calls + 15) // 16, 1, 64
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    pools = [kp.Pool(1, B * maxp, Hkv, d) for _ in streams]
    bt = torch.randperm(B * maxp, device="cuda").to(torch.int32).view(B, maxp).contiguous()
    x = torch.randn(calls, B, Hkv, d, device="cuda").to(torch.bfloat16)
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    note(f"metadata blocks: {calls} appends on {n_streams} streams behind pending work")
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(10):
                torch.mm(busy, busy)
    cu = np.arange(B + 1, dtype=np.int32)
    for c in range(calls):
        k = c % n_streams
        pos = np.full(B, c // n_streams, np.int32)
        kp.kv_append(pools[k], 0, x[c], x[c], bt, pos, cu, stream=streams[k])
    torch.cuda.synchronize()
    for k, pool in enumerate(pools):
        mine = x[k::n_streams]
        n = mine.shape[0]
        kk, vv = kp.kv_gather(pool, 0, bt, np.full(B, n, np.int32))
        assert pool.device_error() == kp.KVP_OK
        want = mine.transpose(0, 1).reshape(B * n, Hkv, d)
        assert torch.equal(kk, want) and torch.equal(vv, want)
        pool.close()
