"""What the sweep of a plain sort or batch leaves to the follow-up: which runs it
reports, and what happens when it reports more than the list holds.  As in
test_gpu_finish.py the route is seen in the control block."""
import numpy as np
import pytest
import torch

import datagen
from test_gpu_finish import (ANY_FINISH, FINISH, GIANT, KINDS, LONG_LEN, LONGER_LEN, PASS_MASK,
                             SLOTS, UNSORTED, batch_checked, clusters, dev, sort_checked)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rs():
    import paper_1511_03404_amd as rs
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rs.lib()
    return rs


def repeated(n, bits, values, copies, seed):
    """Uniform keys, of which `values` keys come `copies` times each.  Their high
    16 bits are spread evenly, so no two of them and few others share those."""
    g = np.random.RandomState(seed)
    k = datagen.keys("uniform", n, bits, seed=seed)
    dt = k.dtype.type
    step = (65536 // values - 1) | 1  # odd: both bytes vary
    v = (np.arange(values).astype(k.dtype) * dt(step) + dt(1)) << dt(bits - 16)
    v |= k[:values] >> dt(16)
    k[g.permutation(n)[:values * copies]] = np.repeat(v, copies)
    return k


# long runs of equal keys beside one that is out of order: only that one is
# looked at again, not those, which a workgroup each would take.  (Of 32-bit keys
# two digits are sorted, and other keys share those with such a run.)
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("pairs", [False, True])
def test_runs_in_order_are_left_alone(rs, oracle_lib, pairs, in_place):
    n, bits, values, keep = 712000, 64, 600, 36
    keys = repeated(n, bits, values, 520, seed=21)
    single = np.flatnonzero(keys == datagen.keys("uniform", n, bits, seed=21))
    at = np.random.RandomState(22).permutation(single)[:100]
    low = keys.dtype.type((1 << (bits - keep)) - 1)
    keys[at] = (keys[at[0]] & ~low) | (keys[at] & low)
    print(f"case pairs={pairs} in_place={in_place}", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs, in_place)
    assert w[FINISH] & 1
    assert w[LONG_LEN] >= values and 1 <= w[UNSORTED] < 8
    assert w[LONGER_LEN] == 0 and w[GIANT] == 0


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("order,descending", [("unsigned", False), ("float", True)])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_more_places_than_the_list_holds(rs, oracle_lib, bits, pairs, order, descending, in_place):
    """Every digit is sorted again.  Of a tile the list holds 64 places, and every
    run out of order makes one at least."""
    n, count, size = 20000, 200, 70
    keys = clusters(n, bits, count, size, 20, seed=23)
    vals = datagen.values(n, bits) if pairs else None
    ctx = rs.Context(0)
    ctx.tune_set(bits, pairs, False, rs.size_class(n), 0)  # 16384 (8192) elements a tile
    tiles = -(-n // (8192 if bits == 64 and pairs else 16384))
    assert count > 64 * tiles
    ws = torch.empty(ctx.workspace_bytes(bits, pairs, n), dtype=torch.uint8, device="cuda")
    kd, vd = dev(keys), dev(vals) if pairs else None
    kw = {"ctx": ctx, "workspace": ws, "order": order, "descending": descending}
    print(f"case bits={bits} pairs={pairs} order={order} in_place={in_place}", flush=True)
    if pairs:
        ko, vo = rs.sort_pairs(kd, vd, *((kd, vd) if in_place else ()), **kw)
    else:
        ko = rs.sort_keys(kd, *((kd,) if in_place else ()), **kw)
    assert ctx.status(ws) == rs.RS_OK
    ok, ov = oracle_lib.sort_ordered(keys, vals, order=order, descending=descending)
    assert np.array_equal(ko.cpu().numpy(), ok), "keys differ"
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov), "values differ"
    w = ws[:256].cpu().numpy().view(np.uint32)
    if order == "unsigned":  # floats' high bits are no even spread: they may take every pass
        assert w[FINISH] & 1 and w[UNSORTED] > 64 * tiles
    ctx.close()


# (64-bit pairs have tiles of 8192 elements and so a longer list)
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("bits,pairs", KINDS[:3])
def test_batch_with_more_places_than_the_list_holds(rs, oracle_lib, bits, pairs, in_place):
    """Every segment that was swept is sorted again."""
    parts = [clusters(20000, bits, 200, 70, 20, seed=s) for s in range(12)]
    parts[3:3] = [datagen.keys("uniform", 30000, bits, seed=1), datagen.keys("uniform", 77, bits),
                  datagen.keys("zero", 20000, bits)]
    keys = np.concatenate(parts)
    off = np.zeros(len(parts) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([p.size for p in parts])
    vals = datagen.values(keys.size, bits) if pairs else None
    ctx = rs.Context(0)
    ctx.tune_set(bits, pairs, True, rs.size_class(keys.size), 0)  # 16384 elements a tile
    ws = torch.empty(ctx.segmented_workspace_bytes(bits, pairs, keys.size, len(parts)),
                     dtype=torch.uint8, device="cuda")
    kd, vd = dev(keys), dev(vals) if pairs else None
    print(f"case bits={bits} pairs={pairs} in_place={in_place}", flush=True)
    ko, vo = rs.segmented_sort(kd, vd, dev(off.view(np.int64)), kd if in_place else None,
                               vd if in_place else None, ctx=ctx, workspace=ws, order="signed",
                               descending=True)
    assert ctx.status(ws) == rs.RS_OK
    ok, ov = oracle_lib.segmented_sort_ordered(keys, vals, off, order="signed", descending=True)
    assert np.array_equal(ko.cpu().numpy(), ok), "keys differ"
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov), "values differ"
    w = ws[:256].cpu().numpy().view(np.uint32)
    assert w[PASS_MASK] & ANY_FINISH
    assert w[UNSORTED] > 64 * (keys.size // 16384 + len(parts) + 1)
    ctx.close()


def giants(n, sizes, keep, seed, clear=0):
    """Uniform 64-bit keys without the bits in `clear`, of which groups of `sizes`
    share their top `keep` bits."""
    g = np.random.RandomState(seed)
    k = datagen.keys("uniform", n, 64, seed=seed)
    at = g.permutation(n)
    low = np.uint64((1 << (64 - keep)) - 1)
    for size in sizes:
        a, at = at[:size], at[size:]
        k[a] = (k[a[0]] & ~low) | (k[a] & low)
    return k & ~np.uint64(clear)


# runs of a tile (16384 elements, 8192 pairs), one more, and several tiles: each is
# sorted by its own lower digits, an odd number of them or an even one
@pytest.mark.parametrize("clear", [0, 0xFF00])
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("order,descending", [("unsigned", False), ("signed", True)])
@pytest.mark.parametrize("pairs", [False, True])
def test_runs_longer_than_a_tile(rs, oracle_lib, pairs, order, descending, in_place, clear):
    tile = 8192 if pairs else 16384
    keys = giants(1 << 22, (tile, tile + 1, 5 * tile // 2, 300), 24, 31, clear)
    print(f"case pairs={pairs} order={order} in_place={in_place} clear={clear}", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs, in_place, order, descending)
    assert w[FINISH] & 1
    # another key may share the first run's 24 bits
    assert w[LONGER_LEN] == 3 and w[GIANT] in (2, 3)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("pairs", [False, True])
def test_segments_with_runs_longer_than_a_tile(rs, oracle_lib, pairs, in_place):
    tile = 8192 if pairs else 16384
    parts = [giants(1 << 22, (tile + 100,), 24, 41), datagen.keys("uniform", 20000, 64, seed=1),
             giants(1 << 22, (tile + 1,), 24, 42, 0xFF0000)]
    print(f"case pairs={pairs} in_place={in_place}", flush=True)
    w = batch_checked(rs, oracle_lib, parts, pairs, in_place, "float", True)
    assert w[LONGER_LEN] == 2 and w[GIANT] == 2


# runs at the edges of what a wave sorts, in four slots and in eight
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_runs_for_a_wave(rs, oracle_lib, bits, pairs, in_place):
    n, sizes = 20000, (65, 128, 255, 256, 257, 511, 512, 513)
    g = np.random.RandomState(51)
    keys = datagen.keys("uniform", n, bits, seed=52)
    at = g.permutation(n)
    low = keys.dtype.type((1 << (bits - 18)) - 1)
    for size in sizes:
        a, at = at[:size], at[size:]
        keys[a] = (keys[a[0]] & ~low) | (keys[a] & low)
        keys[a[:4]] = keys[a[0]]  # equal ones among them, too few for the sample
    print(f"case bits={bits} pairs={pairs} in_place={in_place}", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs, in_place, "signed", True)
    assert w[FINISH] & 1 and w[UNSORTED] >= len(sizes) and 1 <= w[LONGER_LEN] <= 2


# groups of about 19 equal 32-bit keys in one long segment: runs of several groups
# would take the sweep longer than the two passes it saves
@pytest.mark.parametrize("pairs", [False, True])
def test_segment_of_groups_takes_every_digit(rs, oracle_lib, pairs):
    g = np.random.RandomState(61)
    keys = datagen.keys("uniform", 55000, 32, seed=62)[g.randint(0, 55000, 1 << 20)]
    print(f"case pairs={pairs}", flush=True)
    w = batch_checked(rs, oracle_lib, [keys, datagen.keys("uniform", 100, 32)], pairs)
    assert w[PASS_MASK] == 15 and w[LONG_LEN] == 0


# the routes of sorts without long runs, at their edges: the sweep of 32-bit keys in
# a launch of its own (above 2^20), every digit above what two of them leave short
# enough, and the smallest sorts of more than one workgroup
@pytest.mark.parametrize("bits,pairs,n,sweeps", [
    (32, False, (1 << 20) + 77, True), (32, True, (1 << 20) + 77, True),
    (32, False, (1 << 21) + 4095, False), (32, True, (1 << 21) + 4095, False),
    (64, True, 8193, True), (64, False, 16385, True), (32, True, 16385, True)])
def test_route_at_the_edges(rs, oracle_lib, bits, pairs, n, sweeps):
    print(f"case bits={bits} pairs={pairs} n={n}", flush=True)
    w = sort_checked(rs, oracle_lib, datagen.keys("uniform", n, bits, seed=3), pairs)
    assert bool(w[FINISH] & 1) == sweeps and not w[UNSORTED]
    assert (w[SLOTS] < bits // 8) == sweeps
