"""LDS word patterns of the layouts that hold half a tile or less, on the access
geometry measured on gfx950 (profiles/lds_bank_geometry_gfx950.md):

* 4-byte accesses: each half-wave of 32 lanes over 32 banks;
* 16-byte writes: eight consecutive lanes over 32 banks;
* 16-byte reads: sixteen lanes over 64 banks, lanes {0-3, 12-15, 20-23, 24-27}
  and {4-11, 16-19, 28-31} of either half-wave.
"""

import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1306_5076_amd", "csrc")
LANES = np.arange(64)
_FIRST = [0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27]
_SECOND = [x for x in range(32) if x not in _FIRST]
READ_GROUPS = [np.array(g) + h for h in (0, 32) for g in (_FIRST, _SECOND)]
WRITE_GROUPS = [np.arange(8) + 8 * i for i in range(8)]
HALVES = [np.arange(32), np.arange(32) + 32]


def clean(words, width, write):
    """Whether the lanes' accesses at `words` (one per lane) are free of conflicts."""
    words = np.broadcast_to(np.asarray(words), (64,))
    groups, banks = (HALVES, 32) if width == 1 else (WRITE_GROUPS, 32) if write else (READ_GROUPS, 64)
    assert width == 1 or (words % width == 0).all()
    for g in groups:
        at = {int(w) for w in words[g]}  # lanes at one word share it
        if len({(w // width) % (banks // width) for w in at}) != len(at):
            return False
    return True


def test_geometry_model():
    assert clean(LANES, 1, False) and clean(68 * LANES, 4, False) and clean(36 * LANES, 4, True)
    assert not clean(2 * LANES, 1, True) and not clean(8 * LANES, 4, False) and not clean(32 * LANES, 4, True)


def test_colored_sums_stage():
    """bcf_cps.hip: both sides of both directions, by the source's own formula."""
    with open(os.path.join(CSRC, "bcf_cps.hip")) as f:
        place = re.search(r"assume_aligned\(stage, 16\)\) \+ (.*?);\n", f.read()).group(1)
    word = lambda row, q: 4 * eval(place, {"row": row, "q": q})  # noqa: E731
    seen = set()
    for i in range(4):
        shared = word(16 * i + LANES // 4, LANES % 4)  # four lanes per chunk
        own = word(LANES, i)                           # a chunk per lane
        assert clean(shared, 4, True) and clean(own, 4, False)   # loads
        assert clean(own, 4, True) and clean(shared, 4, False)   # stores
        seen |= set(own.tolist())
    assert seen == set(range(0, 1024, 4))


H, HS, S = 32, 36, 68  # kLine / 2, kHalfStride, kLdsStride
SLICE = 2 * 32 * HS     # kHalfLdsWords


@pytest.mark.parametrize("J", [0, 4, 5])
def test_blocked_to_split(J):
    """bcf_device.hpp, blocked_to_split: a 32 x 32 block per half-wave."""
    m, l = SLICE // 2 * (LANES >> 5), LANES & 31
    for c in range(0, H, 4):
        assert clean(m + HS * l + c, 4, True)
    for r in range(H):
        mirror = J > 0 and (r >> (J - 1)) & 1
        words = m + (HS * (r ^ ((1 << (J - 1)) - 1)) + 31 - l if mirror else HS * r + l)
        assert clean(words, 1, False)


@pytest.mark.parametrize("J", [7, 8, 9])
def test_cross_layouts_of_key_groups(J):
    """bcf_device.hpp, keys_to_cross and cross_to_split: half of a group's keys
    at a time in the eight waves' slices."""
    written, read = set(), set()
    for wave in range(8):
        for r in range(0, H, 4):
            w = SLICE * wave + S * (LANES & 31) + H * (LANES >> 5) + r
            assert clean(w, 4, True)
            written |= {int(x) + k for x in w for k in range(4)}
        same, mirror = S * wave + LANES, S * (7 - wave) + 63 - LANES
        for r in range(64):
            up = (r >> (J - 4)) & 1
            src = r ^ ((1 << (J - 4)) - 1) if up else r
            w = (mirror if up else same) + SLICE * (src >> 3) + S * 8 * (src & 3)
            assert clean(w, 1, False)
            read |= set(w.tolist())
    assert read == written  # both halves (bit 2 of src) use the same words
    written, read = set(), set()
    for wave in range(8):
        for r in range(64):
            if (r >> 1) & 1:
                continue
            w = S * wave + LANES + SLICE * (r >> 3) + S * (8 * (r & 1) + 16 * ((r >> 2) & 1))
            assert clean(w, 1, True)
            written |= set(w.tolist())
        for s in range(64):
            if (s >> 4) & 1:
                continue
            w = SLICE * wave + S * 16 * (LANES >> 5) + (LANES & 31) + S * (s & 15) + H * (s >> 5)
            assert clean(w, 1, False)
            read |= set(w.tolist())
    assert read == written


def test_four_wave_tiles():
    """bcf_tile16.hpp, small_wave_clean: words [wave][register][lane], read as
    they are or mirrored."""
    for wave in range(4):
        for r in range(16):
            assert clean(wave * 1024 + 64 * r + LANES, 1, True)
            for other in range(4):
                assert clean(other * 1024 + 64 * r + LANES, 1, False)
                assert clean(other * 1024 + 64 * r + 63 - LANES, 1, False)


def test_u64_merge_tile():
    """bcf_u64.hip, merge_tile64: 2048 keys, a 32-bit half at a time."""
    for r in range(32):
        assert clean(HS * 32 * (LANES >> 5) + (LANES & 31) + HS * (2 * (r % 16) + r // 16), 1, True)
        assert clean(HS * (LANES >> 5) + (LANES & 31) + 2 * HS * r, 1, False)
    for c in range(0, 32, 4):
        assert clean(HS * LANES + c, 4, False) and clean(HS * LANES + c, 4, True)
