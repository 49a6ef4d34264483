"""The block sort of key/value pairs at the edges of its wave tiles (4096) and
group tiles (16384 pairs in four sub-tiles), and the sub-tiles and merge rounds
that a ragged group (pairs or keys) leaves out: bit-exact and stable against
the oracle, on keys full of ties."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 2047, 2049, 4095, 4096, 4097, 8192, 8193, 12289, 16383, 16384, 16385, 40000]


def _keys(n, order):
    rng = np.random.default_rng(n)
    if order == "uniform":
        return rng.integers(0, 1 << 32, n, dtype=np.uint32)
    if order == "ties":
        return rng.choice(np.array([0, 7, 0xFFFFFFFF], dtype=np.uint32), n)
    return np.arange(n, 0, -1, dtype=np.uint32) // 3


@pytest.mark.parametrize("block_sort", [1, 3])
@pytest.mark.parametrize("n", SIZES)
def test_pair_tiles(n, block_sort):
    import torch

    import paper_1306_5076_amd as bcf

    vals = np.random.default_rng(n + 1).integers(0, 1 << 32, n, dtype=np.uint32)
    dv = torch.from_numpy(vals).cuda()
    for order in ("uniform", "ties", "descending"):
        keys = _keys(n, order)
        wk, wv = oracle.sort_pairs_u32(keys, vals)
        with bcf.tuning(block_sort=block_sort):
            ko, vo = bcf.sort_pairs_u32(torch.from_numpy(keys).cuda(), dv)
        assert np.array_equal(ko.cpu().numpy(), wk) and np.array_equal(vo.cpu().numpy(), wv), (order, n)
        ik = keys.view(np.int32)
        idx = np.argsort(ik, kind="stable")
        with bcf.tuning(block_sort=block_sort):
            ko, vo = bcf.sort_pairs_i32(torch.from_numpy(ik).cuda(), dv)
        assert np.array_equal(ko.cpu().numpy(), ik[idx]) and np.array_equal(vo.cpu().numpy(), vals[idx]), (order, n)


@pytest.mark.parametrize("group_min", [1, 4097, 1 << 20])
def test_ragged_groups(group_min):
    import torch

    import paper_1306_5076_amd as bcf

    lengths = np.array(SIZES + [0, 28672, 28673, 32767, 32768, 32769, 65536 + 4097], dtype=np.int64)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    n = int(offs[-1])
    vals = np.random.default_rng(5).integers(0, 1 << 32, n, dtype=np.uint32)
    for order in ("uniform", "ties", "descending"):
        keys = _keys(n, order)
        parts = [oracle.sort_pairs_u32(keys[a:b], vals[a:b]) for a, b in zip(offs[:-1], offs[1:])]
        wk, wv = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
        dk, dv, do = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda(), torch.from_numpy(offs).cuda()
        with bcf.tuning(group_min_keys=group_min):
            got = bcf.segmented_sort(dk, do).cpu().numpy()
            ko, vo = bcf.segmented_sort(dk, do, vals=dv)
        assert np.array_equal(got, wk), order
        assert np.array_equal(ko.cpu().numpy(), wk) and np.array_equal(vo.cpu().numpy(), wv), order
