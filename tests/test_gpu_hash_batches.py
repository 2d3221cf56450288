"""Device chunk hashes around the batches of 16 chunks that the chain takes at a time (whole, and the last, short one), for
every chunk count up to three batches, around eight slabs of 256 leaves and around one to five, with a full and a short last
chunk."""
import numpy as np
import pytest

from oracle.hashing import chunk_hashes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last", [1, 15, 16])
@pytest.mark.parametrize("counts", [list(range(1, 50)), [2031, 2032, 2033, 2047, 2048, 2049, 2063, 2064, 2065]])
def test_chunk_counts_around_the_batches(counts, last):
    import torch
    from paper_2605_06046_amd import fea_chunk_hashes_device
    rng = np.random.default_rng(len(counts) + last)
    lens = [16 * (c - 1) + last for c in counts]
    seqs = [rng.integers(-2 ** 31, 2 ** 31, size=n, dtype=np.int64).astype(np.int32) for n in lens]
    toff = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    hoff = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    sentinel = 0x5A5A5A5A5A5A5A5A
    hashes = torch.full((int(hoff[-1]) + 3,), sentinel, dtype=torch.int64, device="cuda")
    fea_chunk_hashes_device(torch.from_numpy(np.concatenate(seqs)).cuda(), torch.from_numpy(toff).cuda(), torch.from_numpy(hoff).cuda(), hashes)
    torch.cuda.synchronize()
    got = hashes.cpu().numpy().view(np.uint64)
    for i, s in enumerate(seqs):
        assert got[hoff[i]:hoff[i + 1]].tolist() == chunk_hashes(s), counts[i]
    assert (got[hoff[-1]:] == sentinel).all()


@pytest.mark.parametrize("last", [1, 16])
def test_chunk_counts_around_the_slabs(last):
    """Leaves are made 256 at a time, in two buffers in turn; the chain takes them eight at a time out of their lanes."""
    test_chunk_counts_around_the_batches([247, 248, 249, 255, 256, 257, 263, 264, 265, 511, 512, 513, 768, 769, 1025], last)
