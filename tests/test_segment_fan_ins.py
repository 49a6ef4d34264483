"""Merge steps that the host plan of a segmented sort takes by default: the
plan's temp size tells the fan-in, since the tables of both differ."""

import ctypes

import numpy as np
import pytest


def _need(lengths, pairs):
    from paper_1306_5076_amd import _native

    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.uint64)
    need = ctypes.c_uint64(0)
    _native.check("bcf_segmented_upload", _native.load().bcf_segmented_upload(
        off.ctypes.data_as(ctypes.POINTER(ctypes.c_uint64)), len(lengths), pairs, None, ctypes.byref(need), None))
    return need.value


# runs: 4096 below 8192 pairs (16384 keys), else 16384 (32768)
@pytest.mark.parametrize("lengths,pairs,fan_in", [
    ([4097, 8000, 32768, 100], 1, 2), ([20_000] * 300, 1, 2), ([32769, 5000], 1, 4), ([5000, 0, 70_000], 1, 4),
    ([4097, 8000, 65536, 100], 0, 4), ([20_000] * 3355, 1, 2), ([20_000] * 3356, 1, 4),
])
def test_default_fan_in_of_segments(lengths, pairs, fan_in):
    import paper_1306_5076_amd as bcf

    got = _need(lengths, pairs)
    sizes = {}
    for f in (2, 4):
        with bcf.tuning(merge_fan_in=f):
            sizes[f] = _need(lengths, pairs)
    assert sizes[2] != sizes[4]
    assert got == sizes[fan_in]
