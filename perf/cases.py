"""The sorts that a user of this library has it do, as cases that can be timed.

A case is a plain dict:

* ``api``      "sort" (``sort_keys`` / ``sort_pairs``), "segmented"
               (``segmented_sort``) or "merge" (``merge_sort``);
* ``bits``     key width, 32 or 64; ``pairs``: with values (the input index,
               or the index within the segment);
* ``order``    "unsigned", "signed" or "float"; ``descending``;
* ``dist``     how the keys are distributed: the six distributions of the
               benchmark (uniform, gaussian, zero, sorted, reverse, bucket)
               and "ids" (integers below 2^20: the high digits are all zero);
* ``n``        elements of a plain or merge sort;
* ``segments``, ``lo``, ``hi``, ``shape``: a segmented batch of that many
               segments with sizes log-uniform in [lo, hi], drawn from the
               number ``shape``;
* ``kept``     True: the program keeps its output arrays and its workspace
               from call to call, as the benchmark and the serving loop do;
               False: the plain call, which allocates both.
"""
import math

import numpy as np
import torch

import paper_1511_03404_amd as rs

DISTS = ("uniform", "gaussian", "zero", "sorted", "reverse", "bucket", "ids")
IDS_LOG2 = 20


def listed():
    return [
        # the smallest calls: one short list, where latency is all
        _plain("keys32_1000", 1000, 32, False),
        # ranking a list of scores, best first, with their indices
        _plain("scores32_12000", 12000, 32, True, "gaussian", order="float", descending=True),
        # a length of the form 2^k + 2^(k-1), as in the paper's grid; 64-bit ids with row numbers
        _plain("pairs64_98304", 98304, 64, True, "gaussian"),
        # the benchmark's small workload
        _plain("keys32_2p20", 1 << 20, 32, False, kept=True),
        # an odd length of doubles with their indices (an argsort)
        _plain("doubles64_3000017", 3000017, 64, True, "gaussian", order="float"),
        # grouping: few distinct keys, many rows each
        _plain("pairs32_2p24_bucket", 1 << 24, 32, True, "bucket"),
        # the benchmark's 64-bit and main workloads
        _plain("keys64_2p25", 1 << 25, 64, False, kept=True),
        _plain("pairs32_2p26", 1 << 26, 32, True, kept=True),
        # many tiny lists in one call (the benchmark's tiny segments)
        _batch("tiny_lists32", 50000, 2, 1024, 32, True),
        # the benchmark's batch of uneven segments, a tenth of it
        _batch("segments32", 2000, 1 << 4, 1 << 20, 32, True, kept=True),
        # a batch of requests as the serving loop forms it
        _batch("requests64", 24, 1 << 10, 1 << 22, 64, True, kept=True),
        # the merge sort
        _plain("merge32_2p24", 1 << 24, 32, True, api="merge", kept=True),
    ]


def draw(rng):
    api = rng.choice(("sort", "sort", "sort", "segmented", "segmented", "merge"))
    bits = rng.choice((32, 64))
    pairs = rng.random() < 0.6
    order = rng.choice(("unsigned", "unsigned", "signed", "float"))
    dist = rng.choice(DISTS + ("uniform", "uniform", "gaussian"))
    desc = rng.random() < 0.25
    kept = rng.random() < 0.5
    if api == "segmented":
        lo = 1 << rng.randrange(1, 11)
        hi = min(lo << rng.randrange(2, 15), 1 << 22)
        mean = (hi - lo) / math.log(hi / lo)
        most = int((1 << 26) / mean)  # elements in all, on average
        segments = max(1, int(math.exp(rng.uniform(0.0, math.log(max(2, min(most, 200000)))))))
        return _batch("", segments, lo, hi, bits, pairs, dist, order, desc, kept,
                      shape=rng.randrange(1 << 30))
    top = 24 if api == "merge" else 26 if bits == 32 else 25
    n = int(2.0 ** rng.uniform(9, top))
    return _plain("", n, bits, pairs, dist, order, desc, kept, api)


def _plain(name, n, bits, pairs, dist="uniform", order="unsigned", descending=False, kept=False,
           api="sort"):
    c = {"api": api, "n": n, "bits": bits, "pairs": pairs, "dist": dist, "order": order,
         "descending": descending, "kept": kept}
    return {"name": name, **c} if name else c


def _batch(name, segments, lo, hi, bits, pairs, dist="uniform", order="unsigned",
           descending=False, kept=False, shape=1):
    c = {"api": "segmented", "segments": segments, "lo": lo, "hi": hi, "shape": shape,
         "bits": bits, "pairs": pairs, "dist": dist, "order": order, "descending": descending,
         "kept": kept}
    return {"name": name, **c} if name else c


def _sizes(case):
    r = np.random.RandomState(case["shape"])
    lo, hi = math.log(case["lo"]), math.log(case["hi"] + 1)
    s = np.exp(lo + (hi - lo) * r.random_sample(case["segments"])).astype(np.int64)
    return np.clip(s, case["lo"], case["hi"])


def _total(case):
    return int(_sizes(case).sum()) if case["api"] == "segmented" else case["n"]


def _keys(case, n, gen):
    bits, dist = case["bits"], case["dist"]
    dev = "cuda"
    if case["order"] == "float":
        dt = torch.float32 if bits == 32 else torch.float64
        if dist == "zero":
            return torch.zeros(n, dtype=dt, device=dev)
        if dist == "ids":
            return torch.randint(0, 1 << IDS_LOG2, (n,), device=dev, generator=gen).to(dt)
        if dist == "bucket":
            table = torch.randn(64, dtype=dt, device=dev, generator=gen)
            return table[torch.randint(0, 64, (n,), device=dev, generator=gen)]
        if dist == "uniform":
            return torch.rand(n, dtype=dt, device=dev, generator=gen)
        k = torch.randn(n, dtype=dt, device=dev, generator=gen)
        if dist in ("sorted", "reverse"):
            k = torch.sort(k, descending=dist == "reverse").values
        return k
    dt = torch.int32 if bits == 32 else torch.int64

    def words(m):
        w = torch.randint(0, 1 << 32, (m,), device=dev, generator=gen)
        if bits == 32:
            return w
        return (w << 32) | torch.randint(0, 1 << 32, (m,), device=dev, generator=gen)

    def fold(w):  # the low bits of int64 words as keys of the case's width
        if bits == 64:
            return w
        return torch.where(w >= 1 << 31, w - (1 << 32), w).to(dt)

    if dist == "zero":
        return torch.zeros(n, dtype=dt, device=dev)
    if dist == "ids":
        return torch.randint(0, 1 << IDS_LOG2, (n,), device=dev, generator=gen).to(dt)
    if dist == "bucket":
        return fold(words(64))[torch.randint(0, 64, (n,), device=dev, generator=gen)]
    if dist == "gaussian":  # the mean of four uniform draws, each shifted first
        mask = (1 << (bits - 2)) - 1
        s = (words(n) >> 2) & mask
        for _ in range(3):
            s += (words(n) >> 2) & mask
        return fold(s)
    k = words(n)
    if dist in ("sorted", "reverse"):
        k = k ^ (-(1 << 63)) if bits == 64 else k
        k = torch.sort(k, descending=dist == "reverse").values
        k = k ^ (-(1 << 63)) if bits == 64 else k
    return fold(k)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n = _total(case)
    keys = _keys(case, n, gen)
    dt = torch.int32 if case["bits"] == 32 else torch.int64
    offsets = values = None
    if case["api"] == "segmented":
        sizes = torch.from_numpy(_sizes(case)).cuda()
        offsets = torch.zeros(case["segments"] + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(sizes, 0, out=offsets[1:])
    if case["pairs"]:
        values = torch.arange(n, device="cuda")
        if offsets is not None:
            values -= torch.repeat_interleave(offsets[:-1], sizes, output_size=n)
        values = values.to(dt)
    return keys, values, offsets


def prepare(case, seed):
    keys, values, offsets = _inputs(case, seed)
    ctx = rs.context(0)
    kw = {"ctx": ctx, "order": case["order"], "descending": case["descending"]}
    if case["kept"]:
        n, bits, pairs = keys.numel(), case["bits"], case["pairs"]
        if case["api"] == "segmented":
            need = ctx.segmented_workspace_bytes(bits, pairs, n, case["segments"])
        elif case["api"] == "merge":
            need = ctx.merge_workspace_bytes(bits, pairs, n)
        else:
            need = ctx.workspace_bytes(bits, pairs, n)
        kw["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
        if case["api"] == "sort" and not pairs:
            kw["out"] = torch.empty_like(keys)
        else:
            kw["keys_out"] = torch.empty_like(keys)
            if pairs:
                kw["values_out"] = torch.empty_like(values)
    return {"api": case["api"], "keys": keys, "values": values, "offsets": offsets, "kw": kw}


def run(state):
    keys, values, kw = state["keys"], state["values"], state["kw"]
    if state["api"] == "segmented":
        return rs.segmented_sort(keys, values, state["offsets"], **kw)
    if state["api"] == "merge":
        return rs.merge_sort(keys, values, **kw)
    if values is None:
        return rs.sort_keys(keys, **kw)
    return rs.sort_pairs(keys, values, **kw)


def work(case):
    # every key and value read once and written once; a sort does no arithmetic to speak of
    n = _total(case)
    b = 2 * n * (case["bits"] // 8) * (2 if case["pairs"] else 1)
    return {"bytes": b + (8 * (case["segments"] + 1) if case["api"] == "segmented" else 0),
            "flops": 0}


def exact(case, seed):
    keys, values, offsets = _inputs(case, seed)
    if case["order"] == "float":
        k = keys.double()
    else:
        k = keys.long()
        if case["order"] == "unsigned":
            k = k & 0xFFFFFFFF if case["bits"] == 32 else k ^ (-(1 << 63))
    at = torch.sort(k, stable=True, descending=case["descending"]).indices
    del k
    if offsets is not None:
        seg = torch.repeat_interleave(torch.arange(case["segments"], device="cuda"),
                                      offsets[1:] - offsets[:-1], output_size=keys.numel())
        at = at[torch.sort(seg[at], stable=True).indices]
        return keys[at], None if values is None else values[at]
    return keys[at] if values is None else (keys[at], values[at])
