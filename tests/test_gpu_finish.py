"""Plain sorts whose passes stop at a high digit position: the sweep that
orders the runs of equal high bits (k_finish) and what it leaves to k_last.
Every route is forced by the keys and seen in the control block of the
caller's workspace, and every result equals the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import datagen

pytestmark = pytest.mark.gpu

KINDS = [(32, False), (32, True), (64, False), (64, True)]
# words of the control block
FINISH, UNSORTED, LONG_LEN, GIANT, SLOTS, LONGER_LEN = 49, 50, 51, 52, 55, 60


@pytest.fixture(scope="module")
def rs():
    import paper_1511_03404_amd as rs
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rs.lib()
    return rs


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def clusters(n, bits, count, size, keep, seed):
    """Uniform keys, of which `count` groups of `size` share their top `keep`
    bits, spread over the input."""
    g = np.random.RandomState(seed)
    k = datagen.keys("uniform", n, bits, seed=seed)
    at = g.permutation(n)[:count * size].reshape(count, size)
    low = k.dtype.type((1 << (bits - keep)) - 1)
    lead = k[at[:, :1]] & ~low
    k[at] = lead | (k[at] & low)
    return k


def sort_checked(rs, oracle_lib, keys, pairs, in_place=False, order="unsigned", descending=False):
    bits = keys.dtype.itemsize * 8
    vals = datagen.values(keys.size, bits) if pairs else None
    ctx = rs.Context(0)
    ws = torch.empty(ctx.workspace_bytes(bits, pairs, keys.size), dtype=torch.uint8, device="cuda")
    kd, vd = dev(keys), dev(vals) if pairs else None
    kw = {"ctx": ctx, "workspace": ws, "order": order, "descending": descending}
    if pairs:
        ko, vo = rs.sort_pairs(kd, vd, *((kd, vd) if in_place else ()), **kw)
    else:
        ko = rs.sort_keys(kd, *((kd,) if in_place else ()), **kw)
    assert ctx.status(ws) == rs.RS_OK
    if order == "unsigned" and not descending:
        ok, ov = oracle_lib.sort(keys, vals)
    else:
        ok, ov = oracle_lib.sort_ordered(keys, vals, order=order, descending=descending)
    assert np.array_equal(ko.cpu().numpy(), ok), "keys differ"
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov), "values differ"
    words = ws[:256].cpu().numpy().view(np.uint32)
    ctx.close()
    return words


# sizes on both sides of the sweep's tile (2048), one digit more and less,
# the smallest multi-kernel sort
@pytest.mark.parametrize("dist", ["uniform", "gaussian", "sorted", "reverse"])
@pytest.mark.parametrize("n", [16385, 32767, 9 * 2048, 9 * 2048 + 1, (1 << 20) + 77, (1 << 21) + 4095])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_short_runs(rs, oracle_lib, bits, pairs, n, dist):
    print(f"case bits={bits} pairs={pairs} n={n} dist={dist}", flush=True)
    w = sort_checked(rs, oracle_lib, datagen.keys(dist, n, bits, seed=n % 11 + 1), pairs)
    # 32-bit keys take this route only if they save two digits
    if bits == 64 or n < 1 << 20:
        assert w[FINISH] & 1 and not w[UNSORTED]
        assert w[SLOTS] < bits // 8


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("order,descending", [("unsigned", False), ("float", True), ("signed", True)])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_short_runs_orders(rs, oracle_lib, bits, pairs, order, descending, in_place):
    n = 300007 if in_place else 70001
    print(f"case bits={bits} pairs={pairs} order={order} in_place={in_place}", flush=True)
    w = sort_checked(rs, oracle_lib, datagen.keys("uniform", n, bits, seed=5), pairs, in_place,
                     order, descending)
    assert w[FINISH] & 1


# equal keys make long runs that are in order: nothing to do
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_long_runs_in_order(rs, oracle_lib, bits, pairs):
    keys = datagen.keys("uniform", 150001, bits, seed=3)
    keys[::500] = keys[7]
    print(f"case bits={bits} pairs={pairs} equal keys", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs)
    assert w[FINISH] & 1 and w[LONG_LEN] >= 1


# (elements, groups, group size, shared bits): runs on either side of the
# counting limit, of a wave's limit, and one longer than a tile (32-bit keys
# so grouped would be sorted by every digit)
LONG = {
    "run_46": (300007, 3, 46, 20),
    "run_300": (300007, 5, 300, 24),
    "many_runs": (1 << 20, 700, 100, 20),
    "run_1200": (1 << 20, 1, 1200, 24),
    "longer_than_a_tile": (1 << 21, 1, 9000, 24),
}


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("name", sorted(LONG))
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_long_runs_out_of_order(rs, oracle_lib, bits, pairs, name, in_place):
    if name == "longer_than_a_tile" and bits == 32:
        pytest.skip("32-bit keys stop early only when no digit is this uneven")
    n, count, size, keep = LONG[name]
    keys = clusters(n, bits, count, size, keep, seed=17)
    order, desc = ("unsigned", False) if bits == 32 else ("signed", True)
    print(f"case bits={bits} pairs={pairs} {name} in_place={in_place}", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs, in_place, order, desc)
    assert w[FINISH] & 1
    assert bool(w[UNSORTED]) == (name != "run_46")
    assert bool(w[GIANT]) == (name == "longer_than_a_tile")
    assert bool(w[LONGER_LEN]) == (name in ("run_1200", "longer_than_a_tile"))
    if name == "many_runs":
        assert w[LONG_LEN] > 512


# keys in groups of 32 equal ones: runs of several groups, found by the sample
@pytest.mark.parametrize("n", [70001, 1 << 20])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_groups_of_equal_keys(rs, oracle_lib, bits, pairs, n):
    g = np.random.RandomState(4)
    keys = datagen.keys("uniform", n // 32, bits, seed=6)[g.randint(0, n // 32, n)]
    print(f"case bits={bits} pairs={pairs} n={n} groups", flush=True)
    sort_checked(rs, oracle_lib, keys, pairs)


# uneven keys: every digit is sorted, the last one by k_last
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("n", [20001, 500001])
def test_last_pass_in_k_last(rs, oracle_lib, pairs, n, in_place):
    keys = datagen.keys("uniform", n, 64, seed=9)
    keys[np.random.RandomState(1).rand(n) < 0.4] = keys[3]
    print(f"case pairs={pairs} n={n} in_place={in_place}", flush=True)
    w = sort_checked(rs, oracle_lib, keys, pairs, in_place, "float", True)
    assert w[SLOTS] == 8 and not w[FINISH]


def test_graph_replay(rs, oracle_lib):
    """A captured sort whose replays take every route in turn."""
    n = 1 << 20
    inputs = [datagen.keys("uniform", n, 32, seed=2), clusters(n, 32, 5, 300, 24, 3),
              clusters(n, 32, 1, 1200, 24, 4), datagen.keys("bucket", n, 32, seed=5),
              datagen.keys("zero", n, 32)]
    ctx = rs.Context(0)
    keys, vals = dev(inputs[0]), dev(datagen.values(n, 32))
    ws = torch.empty(ctx.workspace_bytes(32, True, n), dtype=torch.uint8, device="cuda")
    ko, vo = torch.empty_like(keys), torch.empty_like(vals)
    rs.sort_pairs(keys, vals, ko, vo, ctx=ctx, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rs.sort_pairs(keys, vals, ko, vo, ctx=ctx, workspace=ws)
    for k in inputs + inputs[:2]:
        keys.copy_(dev(k))
        ko.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ok, ov = oracle_lib.sort(k, datagen.values(n, 32))
        assert np.array_equal(ko.cpu().numpy(), ok) and np.array_equal(vo.cpu().numpy(), ov)
    ctx.close()


PASS_MASK, ANY_FINISH = 49, 1 << 16


def batch_checked(rs, oracle_lib, parts, pairs, in_place=False, order="unsigned",
                  descending=False):
    keys = np.concatenate(parts)
    bits = keys.dtype.itemsize * 8
    off = np.zeros(len(parts) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([p.size for p in parts])
    vals = datagen.values(keys.size, bits) if pairs else None
    ctx = rs.Context(0)
    ws = torch.empty(ctx.segmented_workspace_bytes(bits, pairs, keys.size, len(parts)),
                     dtype=torch.uint8, device="cuda")
    kd, vd = dev(keys), dev(vals) if pairs else None
    ko, vo = rs.segmented_sort(kd, vd, dev(off.view(np.int64)), kd if in_place else None,
                               vd if in_place else None, ctx=ctx, workspace=ws, order=order,
                               descending=descending)
    assert ctx.status(ws) == rs.RS_OK
    ok, ov = oracle_lib.segmented_sort_ordered(keys, vals, off, order=order, descending=descending)
    assert np.array_equal(ko.cpu().numpy(), ok), "keys differ"
    if pairs:
        assert np.array_equal(vo.cpu().numpy(), ov), "values differ"
    words = ws[:256].cpu().numpy().view(np.uint32)
    ctx.close()
    return words


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("order,descending", [("unsigned", False), ("float", True)])
@pytest.mark.parametrize("bits,pairs", KINDS)
def test_segments_of_every_route(rs, oracle_lib, bits, pairs, order, descending, in_place):
    """Large segments side by side whose plans differ: two or more passes and
    the sweep, every digit, one pass fewer, none at all; small ones between."""
    g = np.random.RandomState(8)

    def uni(n, seed):
        return datagen.keys("uniform", n, bits, seed=seed)

    one = uni(40000, 5)
    one[:] = one[0]
    groups = uni(2000, 6)[g.randint(0, 2000, 64000)]
    uneven = uni(50001, 7)
    uneven[g.rand(50001) < 0.4] = uneven[3]
    few = uni(30000, 9) % uni(1, 1).dtype.type(1 << 18)
    parts = [uni(16385, 1), uni(70001, 2), uni(3, 3), one, uni(20000, 4), groups, uneven,
             uni(5000, 8), few, datagen.keys("sorted", 100000, bits, seed=10),
             datagen.keys("gaussian", 300007, bits, seed=11), clusters(300007, bits, 3, 300, 24, 12),
             clusters(400000, bits, 1, 700, 24, 13)]
    print(f"case bits={bits} pairs={pairs} order={order} in_place={in_place}", flush=True)
    w = batch_checked(rs, oracle_lib, parts, pairs, in_place, order, descending)
    assert w[PASS_MASK] & ANY_FINISH
    if order == "unsigned":
        assert w[UNSORTED] and w[LONG_LEN] >= 4


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("pairs", [False, True])
def test_segment_with_a_run_longer_than_a_tile(rs, oracle_lib, pairs, in_place):
    parts = [datagen.keys("uniform", 20000, 64, seed=1), clusters(1 << 23, 64, 1, 17000, 24, 2),
             datagen.keys("gaussian", 60000, 64, seed=3)]
    print(f"case pairs={pairs} in_place={in_place}", flush=True)
    w = batch_checked(rs, oracle_lib, parts, pairs, in_place, "signed", True)
    assert w[GIANT] == 1 and w[LONGER_LEN] >= 1


@pytest.mark.parametrize("bits", [32, 64])
def test_batches_that_do_not_move(rs, oracle_lib, bits):
    parts = [np.full(n, n, dtype=np.uint32 if bits == 32 else np.uint64) for n in (20000, 40001)]
    w = batch_checked(rs, oracle_lib, parts, True)
    assert w[PASS_MASK] == 1 << (bits // 8 - 1)
    batch_checked(rs, oracle_lib, parts, True, in_place=True)
