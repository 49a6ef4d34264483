"""The calls that this library's performance is judged by.

Each case is one call of a public entry point of ``paper_1306_5076_amd`` on data
that is already in device memory, into an output and a workspace that the
program keeps from call to call, as a program that sorts repeatedly does.  The
sizes are those of the benchmark and the tests or lie between them; most are
not powers of two.

Keys are int32 tensors reinterpreted as u32 where the entry point takes u32
keys, and drawn by the device's generator from the seed alone:

  uniform   every bit pattern equally likely (f32: normal deviates)
  zipf      Zipf(1.2) over 2^20 ranks scattered over the key range: a few keys
            make up most of the array
  sorted    uniform keys that are already in order
  few       16 distinct keys
"""

from __future__ import annotations

import numpy as np
import torch

import paper_1306_5076_amd as bcf

_RANKS = 1 << 20
_CDF: dict = {}


def listed():
    return [
        # One short list, sorted once: launch count and the latency of one tile.
        {"name": "keys_3k", "op": "sort", "type": "u32", "n": 3000, "dist": "uniform"},
        # The small configuration of the benchmark: a few tiles and merge passes, still bound by latency.
        {"name": "keys_64k", "op": "sort", "type": "u32", "n": 1 << 16, "dist": "uniform"},
        # An ordinary column of skewed signed keys, with an uneven last tile.
        {"name": "i32_3m_zipf", "op": "sort", "type": "i32", "n": 3_000_017, "dist": "zipf"},
        # The benchmark's main array.
        {"name": "keys_64m", "op": "sort", "type": "u32", "n": 1 << 26, "dist": "uniform"},
        # An argsort of ordinary float keys: the value is the row's index.
        {"name": "pairs_f32_300k", "op": "pairs", "type": "f32", "n": 300_007, "dist": "uniform"},
        # A large stable key/value sort.
        {"name": "pairs_64m", "op": "pairs", "type": "u32", "n": 1 << 26, "dist": "uniform"},
        # 64-bit keys.
        {"name": "u64_12m", "op": "sort", "type": "u64", "n": 12_000_001, "dist": "uniform"},
        # Ten thousand arrays in one call, their offsets in device memory.
        {"name": "segments_10k", "op": "segmented", "pairs": False, "planned": False, "arrays": 10_000, "longest": 1 << 17,
         "dist": "uniform"},
        # Key/value arrays of one fixed layout, planned once and sorted again and again.
        {"name": "segments_pairs", "op": "segmented", "pairs": True, "planned": True, "arrays": 1500, "longest": 1 << 16,
         "dist": "uniform"},
        # A merge of sorted runs of uneven length, their offsets in device memory.
        {"name": "merge_60_runs", "op": "merge", "pairs": False, "runs": 60, "n": 16_000_003, "dist": "uniform"},
        # The sort by distribution on keys with many ties, its pivot buckets on.
        {"name": "distribution_16m", "op": "distribution", "n": 1 << 24, "P": 256, "run_keys": 1 << 18, "dist": "zipf"},
        # Colored prefix sums, half of the most colors.
        {"name": "colors_64m", "op": "colors", "n": 1 << 26, "d": 16},
    ]


def _spread(rng, lo, hi):
    """A size between lo and hi, even over its logarithm; half of them odd."""
    n = int(round(lo * (hi / lo) ** rng.random()))
    return min(hi, max(lo, n | 1 if rng.random() < 0.5 else n))


def draw(rng):
    op = rng.choice(["sort", "sort", "sort", "pairs", "pairs", "segmented", "segmented", "merge", "distribution", "colors"])
    dist = rng.choice(["uniform", "uniform", "zipf", "sorted", "few"])
    if op == "sort":
        kind = rng.choice(["u32", "u32", "i32", "f32", "u64"])
        return {"op": op, "type": kind, "n": _spread(rng, 1000, (1 << 24) if kind == "u64" else (1 << 26)), "dist": dist}
    if op == "pairs":
        return {"op": op, "type": rng.choice(["u32", "i32", "f32"]), "n": _spread(rng, 1000, 1 << 26), "dist": dist}
    if op == "segmented":
        return {"op": op, "pairs": rng.random() < 0.4, "planned": rng.random() < 0.5, "arrays": _spread(rng, 20, 4000),
                "longest": _spread(rng, 1 << 9, 1 << 17), "dist": dist}
    if op == "merge":
        return {"op": op, "pairs": rng.random() < 0.4, "runs": _spread(rng, 2, 1000), "n": _spread(rng, 1 << 16, 1 << 25),
                "dist": dist}
    if op == "distribution":
        return {"op": op, "n": _spread(rng, 1 << 20, 1 << 25), "P": rng.choice([64, 128, 256]),
                "run_keys": rng.choice([1 << 15, 1 << 16, 1 << 18]), "dist": dist}
    return {"op": op, "n": _spread(rng, 1 << 12, 1 << 27), "d": rng.randint(1, 32)}


def _segment_lengths(case):
    """The lengths of the arrays, even over their logarithm from 32 to the longest: the same set for every seed."""
    u = (np.arange(case["arrays"]) + 0.5) / case["arrays"]
    return np.floor(32 * (case["longest"] / 32) ** u).astype(np.int64)


def _offsets(lengths, device=None):
    off = np.zeros(lengths.size + 1, dtype=np.int64)
    np.cumsum(lengths, out=off[1:])
    return off if device is None else torch.from_numpy(off).to(device)


def _size(case):
    return int(_segment_lengths(case).sum()) if case["op"] == "segmented" else case["n"]


def _keys(n, kind, dist, gen):
    """n keys of one type (int32 for u32) on the device."""
    dev = gen.device
    if dist in ("uniform", "sorted"):
        if kind == "f32":
            k = torch.randn(n, generator=gen, device=dev)
        elif kind == "u64":
            k = torch.randint(-(1 << 63), (1 << 63) - 1, (n,), generator=gen, device=dev, dtype=torch.int64)
        else:
            k = torch.randint(-(1 << 31), 1 << 31, (n,), generator=gen, device=dev, dtype=torch.int64).to(torch.int32)
        return _ascending(k, kind) if dist == "sorted" else k
    if dist == "few":
        rank = torch.randint(0, 16, (n,), generator=gen, device=dev, dtype=torch.int64)
    else:
        if dev not in _CDF:
            w = torch.arange(1, _RANKS + 1, dtype=torch.float64, device=dev).pow(-1.2).cumsum(0)
            _CDF[dev] = w / w[-1]
        u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
        rank = torch.searchsorted(_CDF[dev], u).clamp_(max=_RANKS - 1)
    rank *= 2654435761
    if kind == "u64":
        return rank * 0x9E3779B1
    low = rank.to(torch.int32)  # modulo 2^32
    return low.to(torch.float32) if kind == "f32" else low


def _ascending(k, kind):
    """k in the order of its key type, by the plain sort."""
    if kind == "u32":
        return (k ^ -(1 << 31)).sort().values ^ -(1 << 31)
    if kind == "u64":
        return (k ^ -(1 << 63)).sort().values ^ -(1 << 63)
    return k.sort().values


def _values(n, gen):
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=gen, device=gen.device, dtype=torch.int64).to(torch.int32)


def _inputs(case, seed):
    """The arrays of a case: keys, values and offsets, made from the seed."""
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    op, n, s = case["op"], _size(case), {}
    if op == "colors":
        s["values"] = _values(n, gen)
        s["colors"] = torch.randint(0, case["d"], (n,), generator=gen, device=dev, dtype=torch.uint8)
        return s
    kind = case.get("type", "u32")
    s["keys"] = _keys(n, kind, case["dist"], gen)
    if op == "pairs":
        s["vals"] = torch.arange(n, device=dev, dtype=torch.int32)
    elif case.get("pairs"):
        s["vals"] = _values(n, gen)
    if op in ("segmented", "merge"):
        order = np.random.default_rng(int(seed))
        if op == "segmented":
            lengths = order.permutation(_segment_lengths(case))
        else:
            share = order.uniform(0.3, 1.0, case["runs"])
            cut = np.floor(np.cumsum(share) / share.sum() * n).astype(np.int64)
            cut[-1] = n
            lengths = np.diff(cut, prepend=0)
        s["lengths"] = lengths
        s["off"] = _offsets(lengths, dev)
    if op == "merge":  # every run in order
        rows = torch.repeat_interleave(torch.arange(s["lengths"].size, device=dev), s["off"].diff())
        both, _ = ((rows << 32) | (s["keys"].to(torch.int64) & 0xFFFFFFFF)).sort()
        s["keys"] = (both & 0xFFFFFFFF).to(torch.int32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = dict(case)
    s["ws"] = bcf.Workspace()
    if case["op"] == "colors":
        s["out"] = torch.empty_like(s["values"])
        return s
    if case.get("type") == "u64":
        s["keys"] = s["keys"].view(torch.uint64)
    s["out"] = torch.empty_like(s["keys"])
    if "vals" in s:
        s["vout"] = torch.empty_like(s["vals"])
    if case.get("planned"):
        s["plan"] = bcf.SegmentedPlan(_offsets(s["lengths"]), s["keys"].device, pairs=case["pairs"])
    return s


def run(s):
    case, ws = s["case"], s["ws"]
    op, kind = case["op"], case.get("type")
    if op == "sort":
        if kind == "u64":
            return bcf.sort_u64(s["keys"], out=s["out"], workspace=ws).view(torch.int64)
        return getattr(bcf, "sort_" + kind)(s["keys"], out=s["out"], workspace=ws)
    if op == "pairs":
        sort = getattr(bcf, "sort_pairs_" + kind)
        return sort(s["keys"], s["vals"], keys_out=s["out"], vals_out=s["vout"], workspace=ws)
    if op == "segmented":
        if case["planned"]:
            return s["plan"].run(s["keys"], s["out"], s.get("vals"), s.get("vout"))
        return bcf.segmented_sort(s["keys"], s["off"], vals=s.get("vals"), keys_out=s["out"], vals_out=s.get("vout"),
                                  workspace=ws)
    if op == "merge":
        return bcf.merge_runs(s["keys"], s["off"], vals=s.get("vals"), keys_out=s["out"], vals_out=s.get("vout"),
                              workspace=ws)
    if op == "distribution":
        return bcf.sort_u32_pb(s["keys"], P=case["P"], run_keys=case["run_keys"], pivot_buckets=True, out=s["out"],
                               workspace=ws)
    return bcf.colored_prefix_sums(s["values"], s["colors"], case["d"], out=s["out"], workspace=ws)


def work(case):
    """Every input element read once and every output element written once; one addition per element for the sums.
    A comparison sort has no smaller count of operations that the library could not trade for fewer passes."""
    n, op = _size(case), case["op"]
    if op == "colors":
        return {"bytes": 9 * n, "flops": n}
    element = 8 if case.get("type") == "u64" else 4
    if op == "pairs" or case.get("pairs"):
        element += 4
    offsets = 8 * (case["arrays"] + 1) if op == "segmented" else 8 * (case["runs"] + 1) if op == "merge" else 0
    return {"bytes": 2 * element * n + offsets, "flops": 0}


def _u32(x):
    return x.to(torch.int64) & 0xFFFFFFFF


def exact(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op == "colors":
        v, c, out = _u32(s["values"]), s["colors"], torch.zeros(case["n"], dtype=torch.int64, device=s["values"].device)
        for color in range(case["d"]):
            at = (c == color).nonzero().squeeze(1)
            out[at] = v[at].cumsum(0) & 0xFFFFFFFF
        return out.to(torch.int32)
    k, kind = s["keys"], case.get("type", "u32")
    if kind == "u64":
        return _ascending(k, kind)
    if kind == "f32":
        k = k.to(torch.float64)
    elif kind == "u32":
        k = _u32(k)
    if op == "segmented":  # the segment's number above the key
        rows = torch.repeat_interleave(torch.arange(case["arrays"], device=k.device), s["off"].diff())
        k = (rows << 32) | k
    k, order = k.sort(stable=True)
    if kind == "u32":
        k = (k & 0xFFFFFFFF).to(torch.int32)
    elif kind == "i32":
        k = k.to(torch.int32)
    return (k, s["vals"][order]) if "vals" in s else k
