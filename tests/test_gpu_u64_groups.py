"""u64 sorts on either side of the size above which the block sort takes group
tiles of 16384 keys (6 * 2^20): last groups of one to four occupied waves with
a ragged sub-tile, odd and even numbers of merge passes, in place and not;
bit-exact against the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

MOST_TILES = 6 << 20


@pytest.mark.parametrize("n", [MOST_TILES - 1, MOST_TILES, MOST_TILES + 1, MOST_TILES + 4097, MOST_TILES + 2 * 4096,
                               MOST_TILES + 3 * 4096 + 5, MOST_TILES + 16384, (8 << 20) + 2 * 4096 + 77])
def test_u64_block_sort_groups(n):
    import torch

    import paper_1306_5076_amd as bcf

    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 64, n, dtype=np.uint64)
    ties = (keys >> np.uint64(62)) * np.uint64(0x5555555555555555)  # the maximum among them
    falling = np.arange(n, 0, -1, dtype=np.uint64) << np.uint64(30)
    for name, k in (("uniform", keys), ("ties", ties), ("falling", falling)):
        print(f"u64 n={n} {name}", flush=True)
        want = oracle.sort_u64(k)
        t = torch.from_numpy(k).cuda()
        assert np.array_equal(bcf.sort_u64(t).cpu().numpy(), want), (name, n)
        bcf.sort_u64(t, out=t)
        assert np.array_equal(t.cpu().numpy(), want), (name, n)
