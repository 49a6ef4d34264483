"""Merges planned on the device with four-way steps only: jobs of one to four
runs at the edges of the cut steps (1920, 2048, 4096 keys) and of a tile's
halves, copies, in-place merges, and the temp sizes that need no read-back;
bit-exact and stable against the oracle."""

import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

RUNS = [
    [5000], [1, 0], [2048, 2048], [2049, 2047], [4096, 1], [1, 4097], [1919, 1921, 1], [0, 3000, 0, 3000],
    [4095, 0, 0, 0, 4097], [40_000, 3], [3, 40_000], [2048] * 16, [1000] * 17, [8192, 0, 5, 8192, 12_289],
    [70_001, 69_999], [1] * 65,
]


def _case(lengths, kind, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    n = int(off[-1])
    if kind == "ties":
        keys = rng.choice(np.array([0, 9, 0xFFFFFFFF], dtype=np.uint32), n)
    elif kind == "apart":  # every run above the ones after it
        keys = (np.arange(n, 0, -1) * 7).astype(np.uint32)
    else:
        keys = rng.integers(0, 1 << 32, n, dtype=np.uint32)
    for a, b in zip(off[:-1], off[1:]):
        keys[a:b].sort()
    return off, keys, rng.integers(0, 1 << 32, n, dtype=np.uint32)


@pytest.mark.parametrize("case", range(len(RUNS)))
def test_merge_runs_four_way(case):
    import torch

    import paper_1306_5076_amd as bcf

    for kind in ("uniform", "ties", "apart"):
        off, keys, vals = _case(RUNS[case], kind, case)
        wk, wv = oracle.sort_pairs_u32(keys, vals)  # a stable merge of the runs is their stable sort
        do, dk, dv = (torch.from_numpy(x).cuda() for x in (off, keys, vals))
        assert np.array_equal(bcf.merge_runs(dk, do).cpu().numpy(), wk), kind
        ko, vo = bcf.merge_runs(dk, do, vals=dv)
        assert np.array_equal(ko.cpu().numpy(), wk) and np.array_equal(vo.cpu().numpy(), wv), kind
        ko, vo = bcf.merge_runs(dk, do, vals=dv, keys_out=dk, vals_out=dv)
        assert np.array_equal(ko.cpu().numpy(), wk) and np.array_equal(vo.cpu().numpy(), wv), kind


def test_segments_longer_than_the_keys_are_not_touched():
    import torch

    import paper_1306_5076_amd as bcf

    n = 10_000
    keys = torch.randint(0, 1 << 30, (n,), dtype=torch.int32, device="cuda")
    out = torch.full_like(keys, 7)
    ws = bcf.Workspace()
    bcf.sort_u32(torch.zeros(1 << 20, dtype=torch.int32, device="cuda"), workspace=ws)  # a larger workspace
    bcf.segmented_sort(keys, torch.tensor([0, 5000, 3 * n], device="cuda"), keys_out=out, workspace=ws)
    assert bool((out == 7).all())


@pytest.mark.parametrize("pairs", [0, 1])
def test_temp_sizes_equal_the_queries(pairs):
    import torch

    from paper_1306_5076_amd import _native

    lib = _native.load()
    for n, k in ((0, 1), (1, 1), (4097, 3), (1 << 20, 64), (300_001, 1000)):
        off = np.zeros(k + 1, dtype=np.int64)
        off[1:] = n
        d = torch.from_numpy(off).cuda()
        p = ctypes.c_void_p(d.data_ptr())
        a, b = ctypes.c_uint64(), ctypes.c_uint64()
        one = ctypes.c_void_p(1) if pairs else None
        assert lib.bcf_merge_runs(None, one, p, k, None, None, None, ctypes.byref(a), None) == 0
        assert lib.bcf_merge_runs_temp(n, k, pairs, ctypes.byref(b)) == 0 and a.value == b.value
        if pairs:
            assert lib.bcf_segmented_sort_pairs(None, None, None, None, p, k, None, ctypes.byref(a), None) == 0
        else:
            assert lib.bcf_segmented_sort(None, None, p, k, None, ctypes.byref(a), None) == 0
        assert lib.bcf_segmented_sort_temp(n, k, pairs, ctypes.byref(b)) == 0 and a.value == b.value
    assert lib.bcf_segmented_sort_temp(1 << 32, 1, pairs, ctypes.byref(b)) == 1
