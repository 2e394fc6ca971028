"""The bitmask allocator's move from the table of free runs to the flags, as a
lockstep-emulated wave on the CPU: arenas of one node to thousands, against
the oracle, and what the move costs."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

import edge_traces
import emu
import oracle
from paper_2405_07079_amd import workloads as W

NODE = 4096                # granules per node summary


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "emu_take.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", emu.HERE,
                               "-I", emu.CSRC, os.path.join(emu.HERE, "emu_take.cpp"),
                               "-o", so])
        yield ctypes.CDLL(so)


def replay(lib, granules, req, pool, kn, cap_live=4096, with_state=True):
    req = np.ascontiguousarray(req, np.int64)
    res, state = np.full(req.shape, 0x7777, np.int64), np.zeros(4 + 4 * req.size + 2, np.int64)
    sl, status = np.zeros(1, np.int64), np.zeros(1, np.int32)
    moved, steps = ctypes.c_uint32(), ctypes.c_uint64()
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    rc = lib.emu_take_replay(ctypes.c_int64(16 * granules), ctypes.c_int64(16),
                             ctypes.c_int64(req.size), P(req), P(res), P(state) if with_state else None,
                             ctypes.c_int64(state.size), P(sl), P(status), ctypes.c_uint32(pool),
                             ctypes.c_uint32(kn), ctypes.c_uint32(cap_live), ctypes.byref(moved),
                             ctypes.byref(steps))
    assert rc == 0, "node summaries disagree with the flags, or a write past them"
    assert status[0] == 0
    ores, ostate = oracle.replay_heap(W.BITMAP, 16 * granules, 16, req)
    assert np.array_equal(res, ores)
    assert not with_state or np.array_equal(state[:sl[0]], ostate)
    return moved.value, steps.value


def trace(granules, n, seed):
    """Allocations from one granule to an eighth of the arena, frees (some
    partial), so that blocks begin and end anywhere in a node, inside one or
    many nodes apart; then small ones until the pool is outgrown."""
    rng = np.random.default_rng(seed)
    size = np.exp(rng.uniform(0, np.log(max(2, granules / 8)), n)).astype(np.int64)
    nodes = rng.random(n) < 0.2
    size[nodes] = np.maximum(1, size[nodes] // NODE) * NODE
    draw = rng.integers(0, 1 << 32, n)
    cut = np.where(rng.random(n) < 0.3, rng.integers(1, 1 << 31, n), 0)
    req = np.where(rng.random(n) < 0.55, 16 * np.minimum(size, granules), -((cut << 32 | draw) + 1))
    return np.concatenate([req, np.full(120, 16), req[:n // 3]])


# arenas that end on a node, a word, a granule past or before either; more
# nodes than one step of 64; summaries in LDS for one node, three, all
@pytest.mark.parametrize("granules", (NODE, 2 * NODE, 3 * NODE - 1, 3 * NODE + 1, 5 * NODE + 64,
                                      64 * NODE, 65 * NODE + 17, 130 * NODE, 200 * NODE - 63))
@pytest.mark.parametrize("kn", (1, 64))
def test_flags_and_summaries_after_the_move(lib, granules, kn):
    for seed in (1, 2, 3):
        moved, _ = replay(lib, granules, trace(granules, 150, 10 * seed + kn), 768, kn)
        assert moved == 1


def test_the_move_does_not_read_every_node(lib):
    """The same requests on arenas of 64 and of 4,096 nodes: the larger one
    takes a few steps per 64 nodes more, not some for every node."""
    req = np.concatenate([np.full(400, 16), -(np.arange(1, 200) * 7_654_321 + 1),
                          np.full(10, 16)])
    # (no state: writing one reads every node's flags)
    small = replay(lib, 64 * NODE, req, 1024, 64, with_state=False)
    large = replay(lib, 4096 * NODE, req, 1024, 64, with_state=False)
    assert small[0] == large[0] == 1
    assert abs(large[1] - small[1]) < 4096


def test_ragged_arena_on_the_flags(lib):
    """2^20 - 1 granules after the move: blocks that end at the last granule,
    in a ragged last word and node."""
    b = edge_traces.fragments_then_edges(W.BITMAP, (1 << 20) - 1, 16, 300, 120, seed=5)
    moved, _ = replay(lib, (1 << 20) - 1, b.req, 1024, 64)
    assert moved == 1
