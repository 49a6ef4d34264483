"""Device offsets that end a little past the arrays of a call: nothing is
written, neither to the outputs nor behind them.  Every array is a view into a
larger allocation, so that a call that does run past its arrays still stays
inside allocated memory, where the guard words show it."""

import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore:.*past the:RuntimeWarning")]

GUARD = 1 << 16  # words behind every array: more than any of the totals below run past it


def _view(torch, n, fill):
    whole = torch.full((n + GUARD,), fill, dtype=torch.int32, device="cuda")
    return whole, whole[:n]


# (keys, offsets' steps): the capacity of the temp buffers sized for these lies
# up to 1136, 10944 and 33533 keys above their number
@pytest.mark.parametrize("n,k", [(10_000, 4), (65_536, 1000), (3_000_001, 60), (16_000_003, 60)])
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("merge", [False, True])
def test_nothing_is_written_past_the_arrays(n, k, pairs, merge):
    import torch

    import paper_1306_5076_amd as bcf

    whole, keys = _view(torch, n, 0)
    keys.copy_(torch.randint(0, 1 << 30, (n,), dtype=torch.int32, device="cuda"))
    if merge:
        keys.copy_(keys.sort().values)
    ok, out = _view(torch, n, 7)
    vw, vals = _view(torch, n, 3)
    vo, vout = _view(torch, n, 7)
    call = bcf.merge_runs if merge else bcf.segmented_sort
    kw = {"vals": vals, "vals_out": vout} if pairs else {}
    for over in (1, 63, 1000, 30_000):
        off = np.linspace(0, n + over, k + 1).astype(np.int64)
        print(f"n={n} k={k} pairs={pairs} merge={merge} over={over}", flush=True)
        call(keys, torch.from_numpy(off).cuda(), keys_out=out, workspace=bcf.Workspace(), **kw)
        torch.cuda.synchronize()
        assert bool((ok == 7).all()) and bool((vo == 7).all())
        assert bool((whole[n:] == 0).all()) and bool((vw == 3).all())
    # an output shorter than the keys: the shortest array counts
    off = np.linspace(0, n, k + 1).astype(np.int64)
    call(keys, torch.from_numpy(off).cuda(), keys_out=out[:-1], workspace=bcf.Workspace(), **kw)
    assert bool((ok == 7).all()) and bool((vo == 7).all())
    # and offsets that end at the last key are served
    call(keys, torch.from_numpy(off).cuda(), keys_out=out, workspace=bcf.Workspace(), **kw)
    want = keys.clone()
    if not merge:
        for a, b in zip(off[:-1], off[1:]):
            want[a:b] = keys[a:b].sort().values
    assert torch.equal(out, want) and bool((ok[n:] == 7).all()) and bool((vo[n:] == 7).all())
