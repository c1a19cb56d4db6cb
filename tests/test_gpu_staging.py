"""Pinned metadata blocks turned over while the GPU is behind: a block is written again only after the work
that read it, on the null stream (many pieces to a block) and on other streams (a block per call)."""
import numpy as np
import pytest

from gpu_helpers import note
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_streams,calls,behind", [(0, 80, 55), (1, 40, 11), (6, 60, 11)])
def test_metadata_blocks_under_pending_work(n_streams, calls, behind):
    """Each call's page runs take about 190 KB of a 1 MB block (the last quarter's, over 1 MB, replace blocks): the
    calls go through every one of the 12 blocks and wait for the first.  Call c writes every sequence's token at
    position c of its stream's pages; a block handed out too early would give an earlier call a later one's
    positions.  The GPU is still behind at call `behind`, before the first block must be used again."""
    import torch
    B, big, Hkv, d = 8000, 48000, 1, 64
    streams = [torch.cuda.Stream() for _ in range(n_streams)] or [torch.cuda.default_stream()]
    n = len(streams)
    maxp = (calls // n + 15) // 16
    pools = [kp.Pool(1, big * maxp, Hkv, d) for _ in streams]
    bt = torch.randperm(big * maxp, device="cuda").to(torch.int32).view(big, maxp).contiguous()
    x = torch.randn(calls, big, Hkv, d, device="cuda").to(torch.bfloat16)
    busy = torch.randn(4096, 4096, device="cuda")
    size = [B if c < calls - calls // 4 else big for c in range(calls)]
    cu = np.arange(big + 1, dtype=np.int32)
    scratch = kp.Pool(1, B, Hkv, d)
    for s in streams:  # pins the blocks
        for c in range(12 if n_streams else 60):
            kp.kv_append(scratch, 0, x[0][:B], x[0][:B], bt[:B, :1].contiguous() % B, np.zeros(B, np.int32), cu[:B + 1],
                         stream=s)
    torch.cuda.synchronize()
    note(f"metadata blocks: {calls} appends on {n_streams or 'the null'} stream(s) behind pending work")
    done = []
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(60):
                torch.mm(busy, busy)
            done.append(torch.cuda.Event())
            done[-1].record(s)
    for c in range(calls):
        if c == behind:
            assert not any(e.query() for e in done), "the GPU is not behind: the test shows nothing"
        k = c % n
        m = size[c]
        pos = np.full(m, c // n, np.int32)
        kp.kv_append(pools[k], 0, x[c][:m], x[c][:m], bt[:m], pos, cu[:m + 1], stream=streams[k])
    torch.cuda.synchronize()
    for k, pool in enumerate(pools):
        mine = x[k::n]
        first = sum(s == B for s in size[k::n])  # calls that wrote the first B sequences only
        kk, vv = kp.kv_gather(pool, 0, bt, np.full(big, mine.shape[0], np.int32))
        assert pool.device_error() == kp.KVP_OK
        want = mine.transpose(0, 1).clone()
        want[B:, :first] = 0
        want = want.reshape(big * mine.shape[0], Hkv, d)
        assert torch.equal(kk, want) and torch.equal(vv, want)
        pool.close()
    scratch.close()


@pytest.mark.parametrize("stream", [None, 2], ids=["one stream", "hipStreamPerThread"])
def test_threads(stream):
    """Four threads append at once, to pools of their own: on the null stream they share blocks; hipStreamPerThread
    (the handle 2) names another stream in each."""
    import threading
    import torch
    T, calls, B, Hkv, d = 4, 40, 4000, 1, 64
    maxp = (calls + 15) // 16
    pools = [kp.Pool(1, B * maxp, Hkv, d) for _ in range(T)]
    bt = torch.randperm(B * maxp, device="cuda").to(torch.int32).view(B, maxp).contiguous()
    x = torch.randn(T, calls, B, Hkv, d, device="cuda").to(torch.bfloat16)
    cu = np.arange(B + 1, dtype=np.int32)
    torch.cuda.synchronize()
    note(f"metadata blocks: {T} threads, stream {stream}")
    failed = []

    def work(t):
        try:
            for c in range(calls):
                kp.kv_append(pools[t], 0, x[t, c], x[t, c], bt, np.full(B, c, np.int32), cu, stream=stream)
        except Exception as e:  # reported by the test, below
            failed.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(T)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for t, pool in enumerate(pools):
        kk, vv = kp.kv_gather(pool, 0, bt, np.full(B, calls, np.int32))
        assert pool.device_error() == kp.KVP_OK
        want = x[t].transpose(0, 1).reshape(B * calls, Hkv, d)
        assert torch.equal(kk, want) and torch.equal(vv, want)
        pool.close()
