"""Colored prefix sums at the edges of a wave's 2048 elements and of tiles of
several pages, bit-exact against the oracle, with the output in
place and apart."""

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2047, 2048, 2049, 6144, 8192 + 2048, 8192 * 3 - 1, 8192 * 8192 + 4097])
@pytest.mark.parametrize("d", [1, 3, 4, 17])
def test_wave_chunk_edges(n, d):
    import torch

    import paper_1306_5076_amd as bcf

    v, c = workloads.colored_u32(n, d, seed=n % 997 + d)
    want = oracle.colored_prefix_sums(v, c, d)
    tv, tc = torch.from_numpy(v).cuda(), torch.from_numpy(c).cuda()
    for cf in (True, False):
        assert np.array_equal(bcf.colored_prefix_sums(tv, tc, d, conflict_free=cf).cpu().numpy(), want), (n, d, cf)
    bcf.colored_prefix_sums(tv, tc, d, out=tv)
    assert np.array_equal(tv.cpu().numpy(), want), (n, d)
