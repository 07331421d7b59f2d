"""Workspace sizes of batches on the CPU.  A program may size its workspace for
its largest batch, or keep a size from a run before, so neither a smaller batch
nor a newer library may need more."""
import pytest

# (key bits, values, elements, segments, bytes): what these batches have needed
# since the segmented sort's first configurations
PINNED = [
    (64, False, 4675141, 2, 39870464),
    (32, False, 22303217, 72, 95872768),
    (64, True, 88968576, 74, 1517140224),
    (32, True, 6905179, 21144, 321158144),
    (64, True, 12058238, 6, 205524480),
]


@pytest.fixture()
def ctx():
    import paper_1511_03404_amd as rs
    c = rs.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("bits,pairs,total,segments,size", PINNED)
def test_segmented_sizes_kept(ctx, bits, pairs, total, segments, size):
    assert ctx.segmented_workspace_bytes(bits, pairs, total, segments) == size


# the elements at which the batch's histogram chunks double; 4-bit digits have
# little else that grows with the batch
@pytest.mark.parametrize("log2", [24, 25, 26])
@pytest.mark.parametrize("bits,pairs", [(32, False), (64, True)])
def test_larger_batch_needs_no_less(ctx, bits, pairs, log2):
    ctx.tune_set(bits, pairs, True, log2, 1)
    at = ctx.segmented_workspace_bytes(bits, pairs, 1 << log2, 100)
    assert ctx.segmented_workspace_bytes(bits, pairs, (1 << log2) - 1, 100) <= at
