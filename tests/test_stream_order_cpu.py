"""What the streamed forward enqueues, and in which order, without a GPU: the
library runs on a stand-in for the HIP runtime (fake_hip.cpp) that logs every
launch, copy, event record and event wait instead of executing it.

The device copy of the weights that a call's copies write may still be read,
or its memory may still be written, by work that was enqueued on `stream`
before the call, so every copy on the I/O stream has to come after that work;
and a unit's products have to come after the unit's copies."""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2504_15299_amd", "libd2moe.so")

# Runs in a process of its own: the stand-in must come before the runtime.
CHILD = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
I, P, Z = ctypes.c_int32, ctypes.c_void_p, ctypes.c_size_t
class Mwq(ctypes.Structure):
    _fields_ = [(n, I) for n in ("n_experts", "rows", "cols", "group", "b_min", "b_max")] + \
               [(n, P) for n in ("planes", "scales", "zeros")]
class Routing(ctypes.Structure):
    _fields_ = [(n, P) for n in ("logits", "topk_idx", "topk_w", "topk_bits", "hist", "offsets",
                                 "perm", "slot_of", "expert_maxbit", "flags")]
class Unit(ctypes.Structure):
    _fields_ = [(n, I) for n in ("expert", "bits", "load_from", "load_to", "count")]
T, d, f, E, k = 4, 128, 128, 2, 1
HOST = 1 << 30
def mwq(rows, cols, at):
    return Mwq(E, rows, cols, 128, 2, 8, at, at + (1 << 22), at + (2 << 22))
h13, h2 = mwq(2 * f, d, HOST), mwq(d, f, HOST + (4 << 22))
w13, w2 = mwq(2 * f, d, 2 << 30), mwq(d, f, (2 << 30) + (4 << 22))
fake.fake_pinned(P(HOST), P(HOST + int(sys.argv[3])))
r = Routing(*([3 << 30] * 10))
S, IO = P(11), P(12)
ev = (P * 3)(101, 102, 103)
need = Z()
assert L.d2moe_moe_forward_workspace(T, d, f, E, k, 0, ctypes.byref(need)) == 0
hist = (I * (E * 7))()
hist[0], hist[2], hist[7] = 1, 2, 1        # expert 0 at 2 and 4 bits, expert 1 at 2
units = (Unit * 3)(Unit(0, 2, 0, 2, 1), Unit(0, 4, 2, 4, 2), Unit(1, 2, 0, 2, 1))
for call in range(2):
    fake.fake_mark()
    resident = (ctypes.c_uint8 * E)()
    rc = L.d2moe_moe_forward_streamed(P(4 << 30), 1, T, d, f, E, k, ctypes.byref(h13),
                                      ctypes.byref(h2), ctypes.byref(w13), ctypes.byref(w2),
                                      resident, ctypes.byref(r), hist, units, 3, P(5 << 30),
                                      P(6 << 30), need, S, IO, ev)
    assert rc == 0 and list(resident) == [4, 2], (rc, list(resident))
fake.fake_log.restype = ctypes.c_char_p
print(fake.fake_log().decode(), end="")
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


def _two_calls(fake, pinned_bytes):
    """The log of two calls on the same buffers, as (call, op, stream, event)."""
    out = subprocess.run([sys.executable, "-c", CHILD, fake, LIB, str(pinned_bytes)], check=True,
                         capture_output=True, text=True, timeout=60).stdout
    call, log = 0, []
    for line in out.splitlines():
        op, stream, event = line.rsplit(" ", 2)
        if op == "mark":
            call += 1
        else:
            log.append((call, op, int(stream), int(event)))
    return log


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


@pytest.mark.parametrize("pinned_bytes", [1 << 28, 0], ids=["pinned", "pageable"])
def test_copies_wait_for_earlier_work_and_products_for_copies(fake, pinned_bytes):
    log = _two_calls(fake, pinned_bytes)
    before = _ordered_before(log)
    S, IO = 11, 12
    assert {s for _, _, s, _ in log} == {S, IO}

    def is_copy(op):
        return op == "copy" or "copy_delta" in op

    copies = [i for i, e in enumerate(log) if e[2] == IO and is_copy(e[1])]
    work = [i for i, e in enumerate(log) if e[2] == S and e[1].startswith("launch:")]
    per_call = [sum(log[i][0] == c for i in copies) for c in (1, 2)]
    # one launch per unit, or planes and scales of two matrices and the zero
    # points with an expert's first load
    assert per_call == [3, 3] if pinned_bytes else per_call == [16, 16], per_call
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
    log = _two_calls(fake, 1 << 28)
    before = _ordered_before(log)
    for call in (1, 2):
        products = {i for i, e in enumerate(log) if e[0] == call and "gemm" in e[1]}
        for i, e in enumerate(log):
            if e[0] == call and "copy_delta" in e[1]:
                assert not products & before[i]
