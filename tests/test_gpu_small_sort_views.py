"""Small sorts into and from views at every word offset of a 16-byte line (the
tile sort stores 16 bytes at any word), and neither in front of the outputs
nor behind them is anything written."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 4095, 4097, 20_001, 70_003])
@pytest.mark.parametrize("at_in,at_out", [(1, 2), (3, 1), (2, 3), (0, 1), (1, 0)])
def test_views(n, at_in, at_out):
    import torch

    import paper_1306_5076_amd as bcf

    rng = np.random.default_rng(n)
    keys, vals = (rng.integers(0, m, n, dtype=np.uint64).astype(np.uint32) for m in (97, 1 << 32))
    wk, wv = oracle.sort_pairs_u32(keys, vals)

    def view(data, at, fill=7):
        whole = torch.full((n + 64,), fill, dtype=torch.int32, device="cuda")
        if data is not None:
            whole[at:at + n] = torch.from_numpy(data.view(np.int32)).cuda()
        return whole, whole[at:at + n]

    def same(whole, at, want):
        got = whole.cpu().numpy()
        assert np.array_equal(got[at:at + n].view(np.uint32), want)
        assert (got[:at] == 7).all() and (got[at + n:] == 7).all()

    _, k = view(keys, at_in)
    _, v = view(vals, (at_in + 1) % 4)
    ow, o = view(None, at_out)
    vw, vo = view(None, (at_out + 2) % 4)
    bcf.sort_u32(k, out=o)
    same(ow, at_out, wk)
    ow.fill_(7)
    bcf.sort_pairs_u32(k, v, keys_out=o, vals_out=vo)
    same(ow, at_out, wk)
    same(vw, (at_out + 2) % 4, wv)
    kw, k = view(keys, at_in)
    bcf.sort_u32(k, out=k)
    same(kw, at_in, wk)
