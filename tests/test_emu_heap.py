"""One call on a device-resident heap, as a lockstep-emulated wave on the CPU:
the result is published after everything else the call does."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

import emu
import oracle

ALLOC, FREE, DUMP, PARTIAL = 1, 2, 3, 4   # the kernel's operations


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "emu_heap.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", emu.HERE,
                               "-I", emu.CSRC, os.path.join(emu.HERE, "emu_heap.cpp"),
                               "-o", so])
        yield ctypes.CDLL(so)


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_result_is_published_last(lib, algo):
    """At the moment the caller can see a result, the heap's tables and
    registers are those the call leaves; results as the oracle's."""
    A, g = 1 << 16, 64
    o = oracle.Heap(algo, A, g)
    rng = np.random.default_rng(algo)
    ops, want, live = [], [], []
    for i in range(120):
        if live and rng.random() < 0.4:
            x = live.pop(int(rng.integers(len(live))))
            if algo <= 2 and rng.random() < 0.3:
                ops.append((PARTIAL, x + g))
                want.append(o.free_partial(x + g))
            ops.append((FREE, x))
            want.append(o.free(x))
        elif i % 29 == 28:
            ops.append((DUMP, 0))
            want.append(len(o.state()))
        else:
            s = int(rng.integers(2 * g, 4096)) if i % 7 else 2 * A
            off = o.alloc(s)
            ops.append((ALLOC, s))
            want.append(off)
            if off >= 0:
                live.append(off)
    op = np.array([x for x, _ in ops], np.int32)
    arg = np.array([x for _, x in ops], np.int64)
    res, early = np.zeros(len(ops), np.int64), np.zeros(len(ops), np.uint8)
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    lib.emu_heap_calls(ctypes.c_int(algo), ctypes.c_int64(A), ctypes.c_int64(g),
                       ctypes.c_uint32(512), ctypes.c_int64(len(ops)), P(op), P(arg), P(res),
                       P(early))
    assert np.array_equal(res, np.array(want))
    assert not early.any(), f"calls whose result came too soon: {np.nonzero(early)[0][:8]}"
