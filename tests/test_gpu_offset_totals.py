"""What device-planned Python calls make of the last offset: totals that no call
takes raise (with a workspace that holds temp for all the keys and without
one), the temp follows the offsets where they cover few of the keys, and calls
in a graph capture are replayed with the offsets there are."""

import warnings

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _calls(bcf, vals):
    for call in (bcf.merge_runs, bcf.segmented_sort):
        for v in (None, vals):
            yield call, {"vals": v}


@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("steps", [3, 20_000])  # one planner launch checks the offsets, or two
def test_totals_above_32_bits_raise(held, steps):
    import torch

    import paper_1306_5076_amd as bcf

    n = 1 << 16
    keys = torch.zeros(n, dtype=torch.int32, device="cuda")
    vals = torch.zeros_like(keys)
    for call, kw in _calls(bcf, vals):
        ws = bcf.Workspace()
        if held:
            ws.get(1 << 26, keys.device)
        out = torch.full_like(keys, 7)
        for total in (1 << 32, 1 << 40, -1):
            off = torch.zeros(steps + 1, dtype=torch.int64, device="cuda")
            off[-1] = total
            with pytest.raises(bcf.BcfError) as e:
                call(keys, off, keys_out=out, workspace=ws, **kw)
            assert e.value.status == 1
            torch.cuda.synchronize()
            assert bool((out == 7).all())
        # the same workspace serves the next call, and totals past the keys warn
        off[-1] = n
        with warnings.catch_warnings():
            warnings.simplefilter("error")
            call(keys, off, keys_out=out, workspace=ws, **kw)
        assert bool((out == 0).all())
        off[-1] = n + 1
        with pytest.warns(RuntimeWarning, match="past the"):
            call(keys, off, keys_out=out, workspace=ws, **kw)


def test_temp_follows_the_offsets():
    """Offsets that cover a small part of a long tensor: temp for that part."""
    import torch

    import paper_1306_5076_amd as bcf

    n, m = 1 << 25, 50_000
    keys = torch.randint(0, 1 << 30, (n,), dtype=torch.int32, device="cuda")
    keys[:m] = keys[:m].sort().values
    vals = torch.arange(n, dtype=torch.int32, device="cuda")
    host = np.linspace(0, m, 21).astype(np.int64)
    want = oracle.sort_u32(keys[:m].cpu().numpy().view(np.uint32)).view(np.int32)
    for call, kw in _calls(bcf, vals):
        ws = bcf.Workspace()
        out = torch.full_like(keys, 7)
        call(keys, torch.from_numpy(host).cuda(), keys_out=out, workspace=ws, **kw)
        assert ws.buf.numel() < 1 << 22  # temp for all the keys would be more than n * 4 bytes
        assert np.array_equal(out[:m].cpu().numpy(), want) and bool((out[m:] == 7).all())
        # and a workspace that holds temp for all the keys
        ws = bcf.Workspace()
        ws.get(1 << 30, keys.device)
        out.fill_(7)
        call(keys, torch.from_numpy(host).cuda(), keys_out=out, workspace=ws, **kw)
        assert np.array_equal(out[:m].cpu().numpy(), want) and bool((out[m:] == 7).all())


@pytest.mark.parametrize("kept", [False, True])
def test_captured_calls_take_the_offsets_of_each_replay(kept):
    import torch

    import paper_1306_5076_amd as bcf

    n, k = 100_000, 12
    rng = np.random.default_rng(5)
    keys = torch.from_numpy(rng.integers(0, 1 << 31, n).astype(np.int32)).cuda()
    out = torch.empty_like(keys)
    off = torch.from_numpy(np.linspace(0, n, k + 1).astype(np.int64)).cuda()
    ws = bcf.Workspace() if kept else None
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        bcf.segmented_sort(keys, off, keys_out=out, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        bcf.segmented_sort(keys, off, keys_out=out, workspace=ws)
    for r in range(4):
        cut = np.sort(rng.integers(0, n + 1, k - 1))
        host = np.concatenate([[0], cut, [n]]).astype(np.uint64)
        off.copy_(torch.from_numpy(host.astype(np.int64)))
        out.fill_(7)
        g.replay()
        want = oracle.segmented_sort(keys.cpu().numpy().view(np.uint32), host)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want), r
        eager = bcf.segmented_sort(keys, off)
        torch.cuda.synchronize()
        assert torch.equal(eager, out), r


def test_threads_and_streams():
    """Calls of eight threads on streams of their own, behind work that keeps
    the device busy for longer than the host polls at once: each takes its own
    total."""
    import threading

    import torch

    import paper_1306_5076_amd as bcf

    n, k = 40_000, 9
    rng = np.random.default_rng(8)
    host = rng.integers(0, 1 << 31, n).astype(np.int32)
    keys = torch.from_numpy(host).cuda()
    busy = torch.randint(0, 1 << 30, (1 << 25,), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    failed = []

    def work(t):
        try:
            stream, ws, out = torch.cuda.Stream(), bcf.Workspace(), torch.empty_like(keys)
            with torch.cuda.stream(stream):
                for r in range(6):
                    cut = np.linspace(0, n, k + 1 + t).astype(np.int64)
                    off = torch.from_numpy(cut).cuda()
                    bcf.sort_u32(busy)
                    bcf.segmented_sort(keys, off, keys_out=out, workspace=ws)
                    want = oracle.segmented_sort(host.view(np.uint32), cut.astype(np.uint64))
                    if not np.array_equal(out.cpu().numpy().view(np.uint32), want):
                        failed.append((t, r, "keys"))
                    off[-1] = (1 << 32) + t
                    try:
                        bcf.segmented_sort(keys, off, keys_out=out, workspace=ws)
                        failed.append((t, r, "accepted"))
                    except bcf.BcfError:
                        pass
        except Exception as e:  # noqa: BLE001
            failed.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
