"""What the streamed forward enqueues, and in which order, without a GPU.

The device copy of the weights that a call's copies write may still be read,
or its memory may still be written, by work that was enqueued on `stream`
before the call, so every copy on the I/O stream has to come after that work;
and a unit's products have to come after the unit's copies."""
import pytest

import fake_hip

S, IO = fake_hip.STREAM, fake_hip.IO_STREAM


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fake_hip"))


def _two_calls(fake, pinned):
    """Two calls on the same buffers: expert 0 at 2 and 4 bits, expert 1 at 2."""
    call = dict(kind="streamed", T=4, d=128, f=128, E=2, k=1, b_min=2, b_max=8, group=128,
                hist=[[1, 0, 2, 0, 0, 0, 0], [1, 0, 0, 0, 0, 0, 0]],
                units=[(0, 2, 0, 2), (0, 4, 2, 4), (1, 2, 0, 2)], pinned=pinned)
    return fake_hip.calls(fake, [call, call])


def _ordered_before(log):
    """For every entry, the indexes of the entries that are sure to be done
    before it starts."""
    done, recorded, before = {}, {}, []
    for i, (_, op, stream, event) in enumerate(log):
        d = done.setdefault(stream, frozenset())
        if op == "wait":
            d = d | recorded.get(event, frozenset())
        before.append(d)
        done[stream] = d | {i}
        if op == "record":
            recorded[event] = done[stream]
    return before


@pytest.mark.parametrize("pinned", [1 << 39, 0], ids=["pinned", "pageable"])
def test_copies_wait_for_earlier_work_and_products_for_copies(fake, pinned):
    log = _two_calls(fake, pinned)
    before = _ordered_before(log)
    assert {s for _, _, s, _ in log} == {S, IO}

    def is_copy(op):
        return op == "copy" or "copy_delta" in op

    copies = [i for i, e in enumerate(log) if e[2] == IO and is_copy(e[1])]
    work = [i for i, e in enumerate(log) if e[2] == S and e[1].startswith("launch:")]
    per_call = [sum(log[i][0] == c for i in copies) for c in (1, 2)]
    # one launch per unit, or planes and scales of two matrices and the zero
    # points with an expert's first load
    assert per_call == ([3, 3] if pinned else [16, 16])
    first = [i for i in work if log[i][0] == 1]
    assert len(first) >= 7  # two products per unit and the combine
    for c in copies:
        if log[c][0] == 2:
            assert set(first) <= before[c], (log[c], "not after the first call's work")
    # and every copy before the last products that need it
    for call in (1, 2):
        last = max(i for i in work if log[i][0] == call)
        assert {c for c in copies if log[c][0] == call} <= before[last]


def test_copies_overlap_the_products_of_earlier_units(fake):
    """Within a call a later unit's copy does not wait for an earlier unit's
    products."""
    log = _two_calls(fake, 1 << 39)
    before = _ordered_before(log)
    for call in (1, 2):
        products = {i for i, e in enumerate(log) if e[0] == call and "gemm" in e[1]}
        assert products
        for i, e in enumerate(log):
            if e[0] == call and "copy_delta" in e[1]:
                assert not products & before[i]


# Host arrays of the two matrices at the stand-in's addresses: planes, scales and
# zero points of each 64 GiB apart; 2 experts of 128-wide matrices need 64 KiB and
# less each.
_LAST = 5 << 36   # offset of the last array (w2's zero points)


@pytest.mark.parametrize("pinned,by_kernel", [
    (_LAST + 256, True),       # exactly to the end of the last array: 2 x 128 x 1 bytes
    (_LAST + 255, False),      # its last byte is not in the allocation
    (_LAST + 1, False), (_LAST, False), ((2 << 36) + 512, False), (1, False)])
def test_device_reads_host_weights_only_inside_their_allocation(fake, pinned, by_kernel):
    """Weights whose first byte is pinned but that go on past the end of that
    allocation are not read by the device; the runtime copies them, each
    rectangle from wherever it lies."""
    log = _two_calls(fake, pinned)
    ops = {op for _, op, s, _ in log if s == IO}
    assert any("copy_delta" in op for op in ops) == by_kernel
    assert ("copy" in ops) == (not by_kernel)
