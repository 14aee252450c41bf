"""What a pass adds to a context's planned memory: the depth buckets' counts
(two words a cell and one a bucket), the tiles' bitmap rows and their segment
counts, and nothing else that grows with the bucket matrix.  Host only."""
import pytest

from paper_2503_12886_amd import gbr


def grown(counts, size, tile=16):
    """Words of buckets and cells, bitmap rows and 16-bit segment counts of a pass."""
    mfs = max(counts)
    nbk = 64
    while nbk < 8192 and nbk * 8 < mfs:
        nbk *= 2
    nblk = max(1, -(-mfs // 8192))
    row = -(-(-(-mfs // 32)) // 32) * 32
    tiles = len(counts) * (size // tile) ** 2
    bkt, cells = len(counts) * nbk, len(counts) * nbk * nblk
    return 4 * (2 * cells + bkt) + 4 * tiles * row + 2 * tiles * (row // 16)


def planned(counts, size):
    offs = [0]
    for n in counts:
        offs.append(offs[-1] + n)
    # (capacities that do not depend on the counts)
    return gbr.gbr_plan_bytes(16, 64, 16, 200_000, 16 * 64 * 64, 1000, offs, [size] * len(counts), [size] * len(counts))


@pytest.mark.parametrize("big", [9_000, 60_000, 180_000])
def test_uneven_frames(big):
    even, uneven = [600] * 16, [big] + [10] * 15
    assert planned(uneven, 64) - planned(even, 64) == grown(uneven, 64) - grown(even, 64)
