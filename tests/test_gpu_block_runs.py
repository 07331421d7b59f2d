"""One-workgroup sorts of keys whose 16 highest differing bits do not tell them
apart: runs of few distinct keys (ordered one key after another), runs of many
(every digit), and keys that mostly share those bits (every digit at once)."""
import numpy as np
import pytest
import torch

import datagen

pytestmark = pytest.mark.gpu

KINDS = [(32, False), (32, True), (64, False), (64, True)]


@pytest.fixture(scope="module")
def rs():
    import paper_1511_03404_amd as rs
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rs.lib()
    return rs


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def make(name, n, bits, seed):
    g = np.random.RandomState(seed)
    k = datagen.keys("uniform", n, bits, seed=seed)
    dt = k.dtype.type
    low = dt((1 << (bits - 18)) - 1)
    at = g.permutation(n)

    def run(a, keys):  # elements a: `keys` distinct keys that share 18 bits
        if a.size:
            v = (k[a[0]] & ~low) | (datagen.keys("uniform", keys, bits, seed=seed + 1) & low)
            k[a] = v[g.randint(0, keys, a.size)]

    if name == "power_law":  # hashed identifiers, a few of them in most places
        ids = (10 ** (4 * g.rand(n))).astype(np.uint64)
        k = (ids * np.uint64(0x9E3779B97F4A7C15) >> np.uint64(64 - bits)).astype(k.dtype)
    elif name == "groups":  # 32 of each key
        k = k[: max(1, n // 32)][g.randint(0, max(1, n // 32), n)]
    elif name == "peel":  # runs of 2, 3, 40, 64 and 65 keys, next to each other in memory
        for part, keys in zip(np.array_split(at[: n // 2], 5), (2, 3, 40, 64, 65)):
            run(part, keys)
    elif name == "peel_limits":  # just longer than a run ordered by counting
        for a, size in ((0, 65), (100, 66), (200, 128), (400, 129)):
            if n >= 2048:
                run(at[a : a + size], 5)
    elif name == "largest":  # the largest key of all, and the smallest, in such runs
        ones = ~dt(0)
        k[at[: n // 8]] = ones ^ g.randint(0, 2, n // 8).astype(k.dtype)
        k[at[n // 8 : n // 4]] = g.randint(0, 2, n // 4 - n // 8).astype(k.dtype)
    elif name == "many":  # 3% of the elements, all different, in one run
        run(at[: n // 32], 1 << 16)
    elif name == "outlier":  # one key sets the highest bit
        k &= dt((1 << (bits // 2 - 1)) - 1)
        k[n // 2] = dt(1 << (bits - 2))
    elif name == "lognormal":  # amounts: a long tail above most keys
        top = (1 << (bits - 1)) - 1
        k = np.minimum(np.exp(g.randn(n) * 3 + bits * 0.3), top).astype(k.dtype)
    return k


NAMES = ["power_law", "groups", "peel", "peel_limits", "largest", "many", "outlier", "lognormal"]
SIZES = [65, 300, 1000, 1024, 1025, 3000, 4096, 6000, 8192, 8193, 12345, 16383, 16384]


@pytest.mark.parametrize("order,descending", [("unsigned", False), ("signed", True)])
@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_whole_sorts(rs, oracle_lib, bits, pairs, name, order, descending):
    for n in SIZES:
        print(f"case bits={bits} pairs={pairs} {name} n={n} order={order}", flush=True)
        keys = make(name, n, bits, seed=n % 13 + 1)
        vals = datagen.values(n, bits) if pairs else None
        ok, ov = oracle_lib.sort_ordered(keys, vals, order=order, descending=descending)
        kd, vd = dev(keys), dev(vals) if pairs else None
        kw = {"order": order, "descending": descending}
        if pairs:
            ko, vo = rs.sort_pairs(kd, vd, kd, vd, **kw)  # in place
            assert np.array_equal(vo.cpu().numpy(), ov), f"values differ, n={n}"
        else:
            ko = rs.sort_keys(kd, **kw)
        assert np.array_equal(ko.cpu().numpy(), ok), f"keys differ, n={n}"


@pytest.mark.parametrize("tiny_cap", [0, 1024])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_segments_and_merges(rs, oracle_lib, bits, pairs, tiny_cap):
    parts = [make(name, n, bits, seed=n % 7 + 2) for name in NAMES
             for n in (100, 700, 1024, 4000, 4097, 8192)]
    off = np.zeros(len(parts) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([p.size for p in parts])
    keys = np.concatenate(parts)
    vals = datagen.values(keys.size, bits) if pairs else None
    print(f"case bits={bits} pairs={pairs} tiny_cap={tiny_cap}", flush=True)
    ctx = rs.Context(0)
    ctx.tiny_cap(tiny_cap)
    kd, vd = dev(keys), dev(vals) if pairs else None
    ko, vo = rs.segmented_sort(kd, vd, dev(off.view(np.int64)), ctx=ctx)
    ok, ov = oracle_lib.segmented_sort_ordered(keys, vals, off)
    assert np.array_equal(ko.cpu().numpy(), ok)
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov)
    for name in NAMES:  # tiles of 8192
        keys = make(name, 50000, bits, seed=3)
        vals = datagen.values(keys.size, bits) if pairs else None
        out = rs.merge_sort(dev(keys), dev(vals) if pairs else None, ctx=ctx)
        ok, ov = oracle_lib.sort(keys, vals)
        assert np.array_equal((out[0] if pairs else out).cpu().numpy(), ok), name
        if pairs:
            assert np.array_equal(out[1].cpu().numpy(), ov), name
    ctx.close()
