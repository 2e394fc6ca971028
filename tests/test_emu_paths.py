"""Replay paths that change core mid-trace, as lockstep-emulated waves on the
CPU, against the oracle: the bitmask allocator replayed from the lean core's
table of free blocks, continuing on the flags once its pool is too small, and
lean-core heaps continuing on the ordered core."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

import emu
import oracle
from paper_2405_07079_amd import workloads as W


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "emu_paths.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", emu.HERE,
                               "-I", emu.CSRC, os.path.join(emu.HERE, "emu_paths.cpp"),
                               "-o", so])
        yield ctypes.CDLL(so)


def buffers(b, blocks):
    res = np.full(b.req.shape, 0x7777, np.int64)
    lens = np.diff(b.req_off)
    caps = 4 + 2 * blocks(lens) + np.where(b.algo == 3, 64 + lens + 1,
                                           np.where(b.algo == 4, 2048 + lens + 1, 0))
    so = np.zeros(b.heaps + 1, np.int64)
    np.cumsum(caps, out=so[1:])
    return (res, np.zeros(int(so[-1]), np.int64), so, np.zeros(b.heaps, np.int64),
            np.zeros(b.heaps, np.int32), np.zeros(b.heaps, np.uint8))


def bitmap_replay(lib, b, pool, kn=1, cap_live=4096):
    res, state, so, sl, status, moved = buffers(b, lambda n: 2 * n + 1)
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    arena, align = np.ascontiguousarray(b.arena), np.ascontiguousarray(b.align)
    algo, off = np.ascontiguousarray(b.algo, np.int32), np.ascontiguousarray(b.req_off)
    req = np.ascontiguousarray(b.req)
    rc = lib.emu_path_replay(ctypes.c_int64(b.heaps), P(arena), P(align), P(algo), P(off),
                             P(req), P(res), P(state), P(so), P(sl), P(status),
                             ctypes.c_uint32(pool), ctypes.c_uint32(kn),
                             ctypes.c_uint32(cap_live), P(moved))
    assert rc == 0, "node summaries disagree with the flags"
    return res, [state[so[h]:so[h] + sl[h]] for h in range(b.heaps)], status, moved


def check(b, res, states, status):
    ores, ostates, _ = oracle.replay_batch(b)
    for h in range(b.heaps):
        x, y = b.req_off[h], b.req_off[h + 1]
        bad = np.nonzero(res[x:y] != ores[x:y])[0]
        assert bad.size == 0, (f"heap {h} request {bad[0]}: {res[x + bad[0]]}, "
                               f"oracle {ores[x + bad[0]]}")
        assert status[h] == 0
        assert np.array_equal(states[h], ostates[h]), f"heap {h} state"


# the pool holds the tables / is outgrown at once / at some request
@pytest.mark.parametrize("pool,some", ((10240, False), (512, True), (768, True)))
def test_bitmap_from_the_table_of_free_blocks(lib, pool, some):
    rng = np.random.default_rng(pool)
    parts = [W.random_tiny(int(rng.integers(1 << 30)), int(rng.integers(0, 400)), gran,
                           align=int(1 << rng.integers(0, 8)), algo=W.BITMAP,
                           max_granules=max(1, gran // int(rng.integers(1, 40))),
                           p_partial=float(rng.uniform(0, 0.6)))
             for gran in [1, 2, 63, 64, 65, 4095, 4096, 4097]
             + [int(g) for g in rng.integers(1, 12_000, 24)]]
    parts.append(W.uniform_batch(heaps=1, n=1500, algo=W.BITMAP, p_partial=0.1))
    b = W.concat(parts)
    res, states, status, moved = bitmap_replay(lib, b, pool)
    check(b, res, states, status)
    assert moved.any() == some


def test_bitmap_table_edges(lib):
    """An arena of 2^16 granules cut one granule at a time around the rover:
    runs that start right below it, at it and at the arena's end, whole-arena
    blocks, and the live capacity."""
    free = lambda r: -(int(r) + 1)  # noqa: E731
    n, g = 4096, 16
    t = [g] * 5 + [free(0x80000000), free(0), g, 2 * g, (n - 8) * g, g, g, free(0xFFFFFFFF), g,
                   3 * g, n * g] + [free(0)] * 12 + [n * g, g, free(0), (n - 1) * g, g, g,
                                                     free(0x90000000), g, free(0), free(0)]
    b = W.Batch("edges", np.array([n * g]), np.array([g]), np.array([W.BITMAP], np.int32),
                np.array([0, len(t)]), np.array(t, np.int64))
    for pool in (10240, 512):
        check(b, *bitmap_replay(lib, b, pool)[:3])
    b = W.random_tiny(3, 400, 256, align=16, p_alloc=0.8, algo=W.BITMAP, max_granules=4)
    want = emu.replay(b, cf=4096, cl=16, shape=5)
    for pool in (10240, 512):
        res, states, status, _ = bitmap_replay(lib, b, pool, cap_live=16)
        assert status[0] == -4 == want[2][0]
        assert np.array_equal(res, want[0]) and np.array_equal(states[0], want[1][0])


def spill_replay(lib, b, pool, cap_free=4096, cap_live=8192):
    res, state, so, sl, status, moved = buffers(b, lambda n: n + 1)
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    arena, align = np.ascontiguousarray(b.arena), np.ascontiguousarray(b.align)
    algo, off = np.ascontiguousarray(b.algo, np.int32), np.ascontiguousarray(b.req_off)
    req = np.ascontiguousarray(b.req)
    lib.emu_spill_replay(ctypes.c_int64(b.heaps), P(arena), P(align), P(algo), P(off), P(req),
                         P(res), P(state), P(so), P(sl), P(status), ctypes.c_uint32(pool),
                         ctypes.c_uint32(cap_free), ctypes.c_uint32(cap_live), P(moved))
    return res, [state[so[h]:so[h] + sl[h]] for h in range(b.heaps)], status, moved


# TLSF's list heads take 8 KiB of the pool
def spill_pool(algo, bytes_):
    return bytes_ + (8192 if algo == W.TLSF else 0)


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
@pytest.mark.parametrize("pool", (512, 2048))
def test_lean_heap_continues_on_the_ordered_core(lib, algo, pool):
    """The tables outgrow the pool mid-trace, with one chunk of free blocks or
    several: small blocks, partial frees, and the state the class lists were
    left in."""
    n = 5000 if algo == W.TLSF else 2500
    b = W.concat([W.uniform_batch(seed=7, heaps=1, arena=1 << 22, align=16, n=n, p_alloc=0.75,
                                  lo=16, hi=4000, algo=algo, p_partial=0.3),
                  W.uniform_batch(seed=8, heaps=1, n=1200, algo=algo, p_alloc=0.7)])
    res, states, status, moved = spill_replay(lib, b, spill_pool(algo, pool))
    check(b, res, states, status)
    assert moved[0] == 1


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_ordered_continuation_at_capacity(lib, algo):
    """Capacities reached after the move: the same requests are refused and
    the same state is left as on the general core.  With a capacity of 64
    free blocks, a heap that brings more than 48 goes to the general core."""
    b = W.uniform_batch(seed=9, heaps=2, n=1800, algo=algo, p_alloc=0.65)
    for cap in (64, 128):
        want = emu.replay(b, kf=64, kl=64, cf=cap, cl=192, shape=0)
        res, states, status, moved = spill_replay(lib, b, 512, cap_free=cap, cap_live=192) \
            if algo != W.TLSF else spill_replay(lib, b, 8192 + 512, cap_free=cap, cap_live=192)
        assert np.array_equal(res, want[0]) and np.array_equal(status, want[2])
        for h in range(b.heaps):
            assert np.array_equal(states[h], want[1][h])
