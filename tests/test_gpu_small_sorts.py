"""Small sorts under the default tuning (tiles by four waves, merges by ranks)
at the edges of lines, waves, tiles, chunks and fan-ins, bit-exact and stable
against the oracle.  ``gap`` makes one chunk of the first run span every other
run, so that the stretches do not fit the staging area."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 1023, 1024, 1025, 3000, 4095, 4096, 4097, 2 * 4096 + 255, 16 * 4096, 16 * 4096 + 1, 17 * 4096 - 3,
         81 * 4096 + 65, 300_007, (1 << 20) - 1, 1 << 20, (1 << 20) + 1]
ORDERS = ["uniform", "two", "equal", "ascending", "descending", "gap"]


def _keys(order, n):
    rng = np.random.default_rng(n)
    if order == "uniform":
        return rng.integers(0, 1 << 32, n, dtype=np.uint32)
    if order == "two":
        return np.where(rng.random(n) < 0.5, np.uint32(0), np.uint32(0xFFFFFFFF))
    if order == "equal":
        return np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    if order == "gap":
        k = rng.integers(1 << 20, 1 << 30, n, dtype=np.uint32)
        k[:4096][::2] = 3
        k[1:4096][::2] = 0xFFFFFFF0
        return k
    k = np.sort(rng.integers(0, 1 << 32, n, dtype=np.uint32))
    return k if order == "ascending" else k[::-1].copy()


@pytest.mark.parametrize("n", SIZES)
def test_small_sorts(n):
    import torch

    import paper_1306_5076_amd as bcf

    vals = np.random.default_rng(n + 1).integers(0, 1 << 32, n, dtype=np.uint32)
    dv = torch.from_numpy(vals).cuda()
    for order in ORDERS:
        keys = _keys(order, n)
        dk = torch.from_numpy(keys).cuda()
        wk, wv = oracle.sort_pairs_u32(keys, vals)
        assert np.array_equal(bcf.sort_u32(dk).cpu().numpy(), wk), (order, n)
        ko, vo = bcf.sort_pairs_u32(dk, dv)
        assert np.array_equal(ko.cpu().numpy(), wk) and np.array_equal(vo.cpu().numpy(), wv), (order, n)
        ik = keys.view(np.int32)
        idx = np.argsort(ik, kind="stable")
        ko, vo = bcf.sort_pairs_i32(torch.from_numpy(ik).cuda(), dv)
        assert np.array_equal(ko.cpu().numpy(), ik[idx]) and np.array_equal(vo.cpu().numpy(), vals[idx]), (order, n)
        inplace = torch.from_numpy(ik.copy()).cuda()
        bcf.sort_i32(inplace, out=inplace)
        assert np.array_equal(inplace.cpu().numpy(), ik[idx]), (order, n)
