"""Planned key/value segments of one tile each, as many as there are where the
wave tiles' work-groups change between two and four waves: sorted and stable
against the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 5, 511, 512, 513, 515, 1022, 1023, 1024, 1025, 2049])
def test_tiles(tiles):
    import torch

    import paper_1306_5076_amd as bcf

    rng = np.random.default_rng(tiles)
    lengths = rng.integers(1, 300, tiles)
    lengths[rng.integers(0, tiles, 3)] = [4096, 1, 4095]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.uint64)
    n = int(off[-1])
    keys, vals = (rng.integers(0, m, n, dtype=np.uint64).astype(np.uint32) for m in (40, 1 << 32))
    seg = np.repeat(np.arange(tiles), lengths)
    order = np.lexsort((np.arange(n), keys, seg))  # stable, segment by segment
    dk, dv = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()
    plan = bcf.SegmentedPlan(off, dk.device, pairs=True)
    ko, vo = plan.run(dk, torch.empty_like(dk), dv, torch.empty_like(dv))
    assert np.array_equal(ko.cpu().numpy(), keys[order]) and np.array_equal(vo.cpu().numpy(), vals[order])
    wk, wv = oracle.sort_pairs_u32(keys[:int(off[1])], vals[:int(off[1])])
    assert np.array_equal(keys[order][:wk.size], wk) and np.array_equal(vals[order][:wv.size], wv)
