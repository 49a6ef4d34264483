"""The block sort of u32 keys at the edges of its wave tiles (4096 keys: lines
of 64, halves of 2048) and group tiles (32768 keys in eight sub-tiles), bit-exact
against the oracle, with keys that order every merge round differently."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 64, 2047, 2048, 2049, 4095, 4096, 4097, 28672, 32767, 32768, 32769, 65536 + 2049]
ORDERS = ["uniform", "two", "descending", "steps", "maximum"]


def _keys(order, n):
    i = np.arange(n, dtype=np.uint64)
    if order == "uniform":
        return np.random.default_rng(n).integers(0, 1 << 32, n, dtype=np.uint32)
    if order == "two":  # 0-1 keys at the ends of the range
        return np.where(np.random.default_rng(n + 1).random(n) < 0.5, np.uint32(0), np.uint32(0xFFFFFFFF))
    if order == "descending":
        return (np.uint64(0xFFFFFFFF) - i * np.uint64(3)).astype(np.uint32)
    if order == "steps":  # lines, halves and sub-tiles in reverse order of one another
        return (((i ^ np.uint64(0x7FC0)) << np.uint64(8)) & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    return np.where(i % np.uint64(7) == 0, np.uint32(5), np.uint32(0xFFFFFFFF)).astype(np.uint32)


@pytest.mark.parametrize("block_sort", [1, 3])
@pytest.mark.parametrize("n", SIZES)
def test_key_tiles(n, block_sort):
    import torch

    import paper_1306_5076_amd as bcf

    for order in ORDERS:
        keys = _keys(order, n)
        with bcf.tuning(block_sort=block_sort):
            got = bcf.sort_u32(torch.from_numpy(keys).cuda()).cpu().numpy()
        assert np.array_equal(got, oracle.sort_u32(keys)), (order, n)
        # the same bits as int32 keys: the tile is padded with another key
        with bcf.tuning(block_sort=block_sort):
            got = bcf.sort_i32(torch.from_numpy(keys.view(np.int32)).cuda()).cpu().numpy()
        assert np.array_equal(got, np.sort(keys.view(np.int32))), (order, n)
