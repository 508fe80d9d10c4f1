"""The library on a stand-in for the HIP runtime (fake_hip.cpp): what a call
enqueues, without a GPU and without executing any of it.

calls() runs in a process of its own, so that the stand-in comes before the
runtime, a list of calls given as dicts of plain values, and returns what they
enqueued as (call, op, stream, event), with op "launch:<kernel>", "copy",
"record" or "wait"."""
from __future__ import annotations

import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2504_15299_amd", "libd2moe.so")
STREAM, IO_STREAM = 11, 12


def build(folder) -> str:
    so = os.path.join(str(folder), "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


def calls(so: str, specs: list) -> list:
    """Each spec: kind "forward" or "streamed", T, d, f, E, k, b_min, b_max,
    group, and shared_f (8 bits) where there is a shared expert; streamed ones also hist [E][L], units (expert, bits, from, to) and
    pinned, the bytes of host memory from the weights' first that the runtime
    calls pinned."""
    out = subprocess.run([sys.executable, os.path.abspath(__file__), so, LIB, json.dumps(specs)],
                         check=True, capture_output=True, text=True, timeout=120).stdout
    call, log = 0, []
    for line in out.splitlines():
        op, stream, event = line.rsplit(" ", 2)
        if op == "mark":
            call += 1
        else:
            log.append((call, op, int(stream), int(event)))
    return log


def _run(so, lib_path, specs):
    import ctypes
    fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    L = ctypes.CDLL(lib_path)
    I, P, Z = ctypes.c_int32, ctypes.c_void_p, ctypes.c_size_t

    class Mwq(ctypes.Structure):
        _fields_ = [(n, I) for n in ("n_experts", "rows", "cols", "group", "b_min", "b_max")] + \
                   [(n, P) for n in ("planes", "scales", "zeros")]

    class Routing(ctypes.Structure):
        _fields_ = [(n, P) for n in ("logits", "topk_idx", "topk_w", "topk_bits", "hist", "offsets",
                                     "perm", "slot_of", "expert_maxbit", "flags")]

    class Unit(ctypes.Structure):
        _fields_ = [(n, I) for n in ("expert", "bits", "load_from", "load_to", "count")]

    host = 1 << 40
    r = Routing(*([1 << 42] * 10))
    x, out, ws = P(1 << 43), P(2 << 43), P(3 << 43)
    ref = ctypes.byref
    for c in specs:
        fake.fake_mark()
        T, d, f, E, k, b_min, b_max = (c[n] for n in ("T", "d", "f", "E", "k", "b_min", "b_max"))

        def mwq(rows, cols, at, E=E):
            return Mwq(E, rows, cols, c["group"], b_min, b_max, at, at + (1 << 36), at + (2 << 36))

        w13, w2 = mwq(2 * f, d, 1 << 44), mwq(d, f, 2 << 44)
        need, sf = Z(), c.get("shared_f", 0)
        assert L.d2moe_moe_forward_workspace(T, d, f, E, k, sf, ref(need)) == 0
        if c["kind"] == "forward":
            sw13, sw2 = mwq(2 * sf, d, 3 << 44, 1), mwq(d, sf, 4 << 44, 1)
            rc = L.d2moe_moe_forward(x, 1, T, d, f, E, k, ref(w13), ref(w2), ref(r),
                                     ref(sw13) if sf else None, ref(sw2) if sf else None,
                                     8 if sf else 0, sf, out, ws, need, P(STREAM))
            assert rc == 0, rc
            continue
        h13, h2 = mwq(2 * f, d, host), mwq(d, f, host + (3 << 36))
        fake.fake_pinned(P(host), P(host + c["pinned"]))
        hist = (I * (E * (b_max - b_min + 1)))(*[n for row in c["hist"] for n in row])
        units = (Unit * len(c["units"]))(*[
            Unit(e, b, lo, hi, c["hist"][e][b - b_min]) for e, b, lo, hi in c["units"]])
        events = (P * len(units))(*[100 + i for i in range(len(units))])
        resident = (ctypes.c_uint8 * E)()
        rc = L.d2moe_moe_forward_streamed(x, 1, T, d, f, E, k, ref(h13), ref(h2), ref(w13), ref(w2),
                                          resident, ref(r), hist, units, len(units), out, ws, need,
                                          P(STREAM), P(IO_STREAM), events)
        assert rc == 0, rc
    fake.fake_log.restype = ctypes.c_char_p
    print(fake.fake_log().decode(), end="")


if __name__ == "__main__":
    _run(sys.argv[1], sys.argv[2], json.loads(sys.argv[3]))
