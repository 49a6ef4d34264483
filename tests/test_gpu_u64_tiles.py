"""u64 sorts at the edges of the merge passes' tiles (2048 keys) and work-groups
(8192 keys), with keys that split every tile differently between its two runs:
bit-exact against the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4097, 6143, 6145, 8192 + 1, 8192 + 2049, 3 * 8192 - 1, 16384 + 6144, (1 << 19) + 8193, 700_001])
def test_u64_merge_tiles(n):
    import torch

    import paper_1306_5076_amd as bcf

    i = np.arange(n, dtype=np.uint64)
    orders = {
        "uniform": np.random.default_rng(n).integers(0, 1 << 64, n, dtype=np.uint64),
        "ascending": i << np.uint64(31),
        "descending": (np.uint64(n) - i) << np.uint64(33),
        "ties": (i * np.uint64(2654435761) % np.uint64(3)) * np.uint64(0x7FFFFFFFFFFFFFFF),
        "maximum": np.where(i % np.uint64(5) == 0, np.uint64(1), ~np.uint64(0)),
    }
    for name, keys in orders.items():
        got = bcf.sort_u64(torch.from_numpy(keys).cuda()).cpu().numpy()
        assert np.array_equal(got, oracle.sort_u64(keys)), (name, n)


@pytest.mark.parametrize("n", [15, 16, 17, 255, 1023, 1024, 1025, 2049, 4080, 4096 + 17, 8192])
def test_u64_tile_of_four_waves(n):
    import torch

    import paper_1306_5076_amd as bcf

    rng = np.random.default_rng(n)
    for keys in (rng.integers(0, 1 << 64, n, dtype=np.uint64), rng.integers(0, 3, n, dtype=np.uint64) << np.uint64(62),
                 np.arange(n, 0, -1, dtype=np.uint64) << np.uint64(30), np.full(n, ~np.uint64(0), dtype=np.uint64)):
        want = oracle.sort_u64(keys)
        t = torch.from_numpy(keys).cuda()
        assert np.array_equal(bcf.sort_u64(t).cpu().numpy(), want), n
        bcf.sort_u64(t, out=t)
        assert np.array_equal(t.cpu().numpy(), want), n
