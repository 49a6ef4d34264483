"""Passes over the data that sorts make: rank passes of small sorts counted as
they are, and as many launches as the count says."""

import pytest

SMALL = {0: 1 << 19, 1: 1 << 20}


@pytest.mark.parametrize("pairs", [0, 1])
def test_counts(pairs):
    import paper_1306_5076_amd as bcf

    want = {0: 0, 1: 1, 4096: 1, 4097: 2, 3 * 4096: 2, 1 << 16: 2, (1 << 16) + 1: 3, SMALL[pairs]: 3}
    assert {n: bcf.sort_data_passes(n, pairs) for n in want} == want
    for n in (SMALL[pairs] + 1, 1 << 24, 1 << 26):
        assert bcf.sort_data_passes(n, pairs) == bcf.sort_passes(n, pairs)
    for knobs in ({"merge_fan_in": 2}, {"merge_fan_in": 4}, {"block_sort": 2}, {"merge_variant": 1},
                  {"fused_partition": 0}, {"tile_samples": 0}, {"sampled_partition": 0}):
        with bcf.tuning(**knobs):
            for n in want:
                assert bcf.sort_data_passes(n, pairs) == bcf.sort_passes(n, pairs), (knobs, n)


@pytest.mark.gpu
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("n", [4096, 20_000, 1 << 16, (1 << 16) + 1, 1 << 19])
def test_launches(n, pairs):
    import torch

    import paper_1306_5076_amd as bcf

    k = torch.randint(0, 1 << 30, (n,), dtype=torch.int32, device="cuda")
    bcf.profile_collect()
    bcf.profile_enable(True)
    try:
        bcf.sort_pairs_u32(k, k) if pairs else bcf.sort_u32(k)
        st = bcf.profile_collect()
    finally:
        bcf.profile_enable(False)
    assert sum(s["launches"] for s in st.values()) == bcf.sort_data_passes(n, pairs), st
