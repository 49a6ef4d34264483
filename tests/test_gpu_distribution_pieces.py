"""The distribution's scatter where an output tile holds a few pieces (walked),
many (each key finds its own) or more than a work-group stages, with empty
ones between them: keys, offsets and splitters bit-exact against the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pb", [False, True])
@pytest.mark.parametrize("n,s,P", [(100_003, 64, 64), (60_000, 16, 8), (20_011, 64, 64), (9000, 200, 64), (300_000, 9, 40),
                                   (4096, 33, 2), (70_000, 64, 256)])
def test_scatter_pieces(n, s, P, pb):
    import torch

    import paper_1306_5076_amd as bcf

    rng = np.random.default_rng(n + s)
    cut = np.sort(rng.integers(0, n + 1, s - 1))
    off = np.concatenate([[0], cut, [n]]).astype(np.uint64)
    for top in (1 << 32, 50):  # distinct keys, and runs full of ties (empty pieces)
        keys = rng.integers(0, top, n, dtype=np.uint64).astype(np.uint32)
        for a, b in zip(off[:-1], off[1:]):
            keys[int(a):int(b)].sort()
        out, pieces, spl = bcf.distribute_runs(torch.from_numpy(keys).cuda(), off, P, P, pivot_buckets=pb)
        want = oracle.distribute_runs(keys, off, P, P, pb)
        assert np.array_equal(out.cpu().numpy(), want[0]), (n, s, P, pb, top)
        assert np.array_equal(pieces.cpu().numpy().astype(np.uint64), want[1])
        assert np.array_equal(spl.cpu().numpy(), want[2])
