"""Sorts that one workgroup or one wave holds (up to 16384 elements), whole or as segments:
every shape at its edges, and keys for every way through it: the 16 highest
differing bits at any place in the key, runs of equal high bits within the
counting limit, beyond it in order, and beyond it out of order."""
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
    if name == "high_run":  # a long run of equal high bits, out of order
        at = g.permutation(n)[: max(2, n // 3)]
        low = dt((1 << (bits - 20)) - 1)
        k[at] = (k[at[0]] & ~low) | (k[at] & low)
    elif name == "two_keys_run":  # two keys, many of each, in one run out of order
        at = g.permutation(n)[: max(2, n // 3)]
        k[at] = k[at[0]] ^ (g.randint(0, 2, at.size).astype(k.dtype) << dt(bits // 4))
    elif name == "equal_run":  # the same, but all its keys equal
        k[g.permutation(n)[: max(2, n // 3)]] = k[0]
    elif name == "mid_bits":  # differing bits 17..34 (64-bit) or 5..21, ones above
        lo, hi = (17, 35) if bits == 64 else (5, 22)
        m = dt(((1 << hi) - 1) & ~((1 << lo) - 1))
        k = (k & m) | ~dt((1 << hi) - 1)
    elif name == "top_byte_and_low":  # 16 high bits that take few values
        k &= dt((0xC0 << (bits - 8)) | 0xFFF)
    elif name == "small":  # below 200: one pass
        k %= dt(200)
    elif name == "one":
        k[:] = k[0]
    return k


NAMES = ["uniform", "high_run", "two_keys_run", "equal_run", "mid_bits", "top_byte_and_low", "small", "one"]
SIZES = [2, 65, 1024, 1025, 2048, 2049, 4095, 4097, 8192, 8193, 16384]


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_whole_sorts(rs, oracle_lib, bits, pairs, name):
    for n in SIZES:
        print(f"case bits={bits} pairs={pairs} {name} n={n}", flush=True)
        keys = make(name, n, bits, seed=n % 13 + 1)
        vals = datagen.values(n, bits) if pairs else None
        ok, ov = oracle_lib.sort(keys, vals)
        kd, vd = dev(keys), dev(vals) if pairs else None
        if pairs:
            ko, vo = rs.sort_pairs(kd, vd, kd, vd)  # in place
            assert np.array_equal(vo.cpu().numpy(), ov), f"values differ, n={n}"
        else:
            ko = rs.sort_keys(kd)
        assert np.array_equal(ko.cpu().numpy(), ok), f"keys differ, n={n}"


@pytest.mark.parametrize("tiny_cap", [0, 1024])
@pytest.mark.parametrize("order,descending", [("unsigned", False), ("float", True)])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_segments(rs, oracle_lib, bits, pairs, order, descending, tiny_cap):
    """The same keys as segments of one batch: without the tiny class, and as
    tiny segments (one wave each) at the edges of its shapes."""
    sizes = (2, 64, 65, 255, 256, 257, 512, 513, 1000, 1024) if tiny_cap else (2, 700, 4096, 4097, 8192)
    parts = [make(name, n, bits, seed=n % 7 + 2) for name in NAMES for n in sizes]
    off = np.zeros(len(parts) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([p.size for p in parts])
    keys = np.concatenate(parts)
    vals = datagen.values(keys.size, bits) if pairs else None
    print(f"case bits={bits} pairs={pairs} order={order}", flush=True)
    ctx = rs.Context(0)
    ctx.tiny_cap(tiny_cap)
    ko, vo = rs.segmented_sort(dev(keys), dev(vals) if pairs else None, dev(off.view(np.int64)),
                               ctx=ctx, order=order, descending=descending)
    ok, ov = oracle_lib.segmented_sort_ordered(keys, vals, off, order=order, descending=descending)
    assert np.array_equal(ko.cpu().numpy(), ok)
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov)
    ctx.close()


@pytest.mark.parametrize("bits,pairs", KINDS)
def test_batches_of_one_class(rs, oracle_lib, bits, pairs):
    """Batches whose total is at the edge of a size class, as one segment and
    cut in two: the launches of the longer classes are left out."""
    for total in (1, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385):
        for cut in (0, total // 3):
            print(f"case bits={bits} pairs={pairs} total={total} cut={cut}", flush=True)
            keys = make("uniform", total, bits, seed=total % 17)
            vals = datagen.values(total, bits) if pairs else None
            off = np.array([0, cut, total], dtype=np.uint64)
            ko, vo = rs.segmented_sort(dev(keys), dev(vals) if pairs else None,
                                       dev(off.view(np.int64)))
            ok, ov = oracle_lib.segmented_sort_ordered(keys, vals, off, order="unsigned",
                                                       descending=False)
            assert np.array_equal(ko.cpu().numpy(), ok)
            if pairs:
                assert np.array_equal(vo.cpu().numpy(), ov)
