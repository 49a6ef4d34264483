"""Planned key/value segments of at most two runs, and of three: sorted and
stable against the oracle, and again after other inputs."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[4097, 8191, 8192, 16385, 32768, 1, 0, 4096], [16384, 16385], [8191] * 40, [32769, 5000]])
def test_planned_pairs(lengths):
    import torch

    import paper_1306_5076_amd as bcf

    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.uint64)
    n = int(off[-1])
    plan = bcf.SegmentedPlan(off, torch.device("cuda", 0), pairs=True)
    for seed, top in ((1, 50), (2, 1 << 32)):
        rng = np.random.default_rng(seed)
        keys, vals = (rng.integers(0, m, n, dtype=np.uint64).astype(np.uint32) for m in (top, 1 << 32))
        dk, dv = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()
        ko, vo = plan.run(dk, torch.empty_like(dk), dv, torch.empty_like(dv))
        hk, hv = bcf.segmented_sort(dk, off, vals=dv, keys_out=dk, vals_out=dv)
        for a, b in zip(off[:-1].astype(int), off[1:].astype(int)):
            wk, wv = oracle.sort_pairs_u32(keys[a:b], vals[a:b])
            for k, v in ((ko, vo), (hk, hv)):
                assert np.array_equal(k[a:b].cpu().numpy(), wk) and np.array_equal(v[a:b].cpu().numpy(), wv), (a, b)
