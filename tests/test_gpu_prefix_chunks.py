"""Block hashing and prefix lookup where a sequence's 64-page chunks fill a wave, a workgroup's pass and more,
and where the first miss falls on the first, last or only page of a chunk."""
import numpy as np
import pytest

from gpu_helpers import note
from oracle import prefix_hash as PH
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pages", [[64 * 64], [64 * 64 + 1, 1, 63], [1024 * 64], [1024 * 64 + 65, 0, 130]])
def test_hashes_and_lookup_over_many_chunks(pages):
    import torch
    rng = np.random.default_rng(sum(pages))
    lens = [16 * n + (7 if i % 2 else 0) for i, n in enumerate(pages)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = rng.integers(0, 151936, size=int(cu[-1]), dtype=np.int64).astype(np.int32)
    note(f"hashes over {pages} pages")
    got = kp.kvp_block_hashes(torch.from_numpy(t).cuda(), cu, seed=11)
    ref = [np.array(PH.block_hashes(t[cu[i]:cu[i + 1]], 11), dtype=np.uint64) for i in range(len(pages))]
    assert np.array_equal(got.cpu().numpy().view(np.uint64), np.concatenate(ref))
    off = kp.block_hash_offsets(cu)
    for miss in (0, 1, 63, 64, 127, 4095, 4096, 65535, 65536, 1 << 30):  # the page of each sequence left out
        table = kp.PrefixTable(18)
        ids = torch.arange(got.numel(), dtype=torch.int32, device="cuda")
        keep = torch.ones(got.numel(), dtype=torch.bool, device="cuda")
        for i, n in enumerate(pages):
            if miss < n:
                keep[int(off[i]) + miss] = False
        table.insert(got[keep].contiguous(), ids[keep].contiguous())
        matched, out = table.lookup(got, cu)
        assert table.error() == kp.KVP_OK
        for i, n in enumerate(pages):
            m = min(miss, n)
            assert int(matched[i]) == m
            row = out[int(off[i]):int(off[i + 1])]
            assert torch.equal(row[:m], ids[int(off[i]):int(off[i]) + m]) and bool((row[m:] == -1).all())
        table.close()
