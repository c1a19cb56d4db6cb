"""Block hashing and prefix lookup of calls with a long sequence, which take a pass of their own: one chunk below,
at and above the lines (256 chunks for the hashes, 1536 for the lookup), a last chunk of one page, more chunks than a
workgroup takes at once, short and empty sequences beside them."""
import numpy as np
import pytest

from gpu_helpers import note
from oracle import prefix_hash as PH
from paper_2608_11152_amd import kvpattn as kp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pages", [[255 * 64 + 63], [256 * 64], [256 * 64 + 1], [257 * 64 + 2, 0, 1, 64, 65],
                                   [3, 1536 * 64, 0], [1536 * 64 + 1, 130], [5, 4096 * 64 + 65, 0, 300 * 64]])
def test_long_sequences(pages):
    import torch
    rng = np.random.default_rng(sum(pages))
    lens = [16 * n + (7 if i % 2 else 0) for i, n in enumerate(pages)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = rng.integers(0, 151936, size=int(cu[-1]), dtype=np.int64).astype(np.int32)
    note(f"hashes of long sequences, {pages} pages")
    got = kp.kvp_block_hashes(torch.from_numpy(t).cuda(), cu, seed=5)
    ref = [np.array(PH.block_hashes(t[cu[i]:cu[i + 1]], 5), dtype=np.uint64) for i in range(len(pages))]
    assert np.array_equal(got.cpu().numpy().view(np.uint64), np.concatenate(ref))
    off = kp.block_hash_offsets(cu)
    ids = torch.arange(got.numel(), dtype=torch.int32, device="cuda")
    last = max(pages) - 1
    for miss in (0, 64, 4095, 65536 + 63, 1536 * 64, 4096 * 64 - 1, 4096 * 64, last, 1 << 30):  # the pages left out
        table = kp.PrefixTable(21)
        keep = torch.ones(got.numel(), dtype=torch.bool, device="cuda")
        for i, n in enumerate(pages):
            for p in (miss, miss + 1000):  # and one behind the first
                if p < n:
                    keep[int(off[i]) + p] = False
        table.insert(got[keep].contiguous(), ids[keep].contiguous())
        matched, out = table.lookup(got, cu)
        assert table.error() == kp.KVP_OK
        for i, n in enumerate(pages):
            m = min(miss, n)
            assert int(matched[i]) == m
            row = out[int(off[i]):int(off[i + 1])]
            assert torch.equal(row[:m], ids[int(off[i]):int(off[i]) + m]) and bool((row[m:] == -1).all())
        table.close()
