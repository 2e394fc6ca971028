"""Where a heap goes when it leaves the lean core, as lockstep-emulated waves
on the CPU: the early hand-over to the ordered core at every size of table,
against the oracle."""
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

LEAN, ORDERED = 0, 1       # (2: the general core)
NOMETA = -4
# ReplayParams::lean_early: the main launch's rule, the heavy launch's rule
MAIN, HEAVY = 1, 2
LIMIT = {0: 256, 1: 384, 2: 1024, 3: 512, 4: 512}   # lean_max_free


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "emu_moves.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", emu.HERE,
                               "-I", emu.CSRC, os.path.join(emu.HERE, "emu_moves.cpp"),
                               "-o", so])
        yield ctypes.CDLL(so)


def replay(lib, b, pool, early, cap_free=4096, cap_live=8192):
    lens = np.diff(b.req_off)
    caps = 4 + 2 * (lens + 1) + np.where(b.algo == 3, 64 + lens + 1,
                                         np.where(b.algo == 4, 2048 + lens + 1, 0))
    so = np.zeros(b.heaps + 1, np.int64)
    np.cumsum(caps, out=so[1:])
    res, state = np.full(b.req.shape, 0x7777, np.int64), np.zeros(int(so[-1]), np.int64)
    sl, status = np.zeros(b.heaps, np.int64), np.zeros(b.heaps, np.int32)
    nxt = np.zeros(b.heaps, np.int32)
    at, free = np.zeros(b.heaps, np.int64), np.zeros(b.heaps, np.int64)
    P = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    arena, align = np.ascontiguousarray(b.arena), np.ascontiguousarray(b.align)
    algo, off = np.ascontiguousarray(b.algo, np.int32), np.ascontiguousarray(b.req_off)
    req = np.ascontiguousarray(b.req)
    lib.emu_move_replay(ctypes.c_int64(b.heaps), P(arena), P(align), P(algo), P(off), P(req),
                        P(res), P(state), P(so), P(sl), P(status), ctypes.c_uint32(pool),
                        ctypes.c_int(early), ctypes.c_uint32(cap_free),
                        ctypes.c_uint32(cap_live), P(nxt), P(at), P(free))
    return res, [state[so[h]:so[h] + sl[h]] for h in range(b.heaps)], status, nxt, at, free


def fragments(algo, f, more=200, seed=1):
    """One heap that comes to about 1.1 f free blocks: 4.4 f small blocks, a
    random half of them freed (half of those next to another), then a mix."""
    rng = np.random.default_rng(seed)
    n = int(4.4 * f)
    k = int(2.2 * f)
    draw = lambda m: -(rng.integers(0, 1 << 32, m) + 1)  # noqa: E731
    size = lambda m: rng.integers(1, 5, m) * 16          # noqa: E731
    mix = np.where(rng.random(more) < 0.5, size(more), draw(more))
    req = np.concatenate([size(n), draw(k), mix]).astype(np.int64)
    return W.Batch("fragments", np.array([1 << 22]), np.array([16]),
                   np.array([algo], np.int32), np.array([0, req.size]), req)


def check_oracle(b, res, states, status):
    ores, ostates, _ = oracle.replay_batch(b)
    assert np.array_equal(res, ores) and (status == 0).all()
    for h in range(b.heaps):
        assert np.array_equal(states[h], ostates[h]), f"heap {h} state"


def check_refused(b, res, states, status):
    """As the oracle on the trace without the requests that met a capacity
    (each changed nothing)."""
    assert (status[0] == NOMETA) == (res == NOMETA).any() and status[0] in (0, NOMETA)
    taken, left = edge_traces.without_refused(b, res, NOMETA)
    check_oracle(taken, left, states, np.zeros(1, np.int32))


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
@pytest.mark.parametrize("early", (MAIN, HEAVY))
def test_early_hand_over_to_the_ordered_core(lib, algo, early):
    """Past the limit the heap goes on to the ordered core between two blocks
    of requests, with its pool far from full."""
    b = fragments(algo, LIMIT[algo] + 120)
    res, states, status, nxt, at, free = replay(lib, b, 61440, early)
    check_oracle(b, res, states, status)
    assert nxt[0] == ORDERED and at[0] % 64 == 0
    assert LIMIT[algo] < free[0] <= LIMIT[algo] + 64


# capacities around the limit: one below it, one where the ordered core takes
# fewer free blocks than the limit, and the first where it takes enough
@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_hand_over_never_ends_on_the_general_core(lib, algo):
    """A pool that holds the tables: the heap stays on the lean core (main
    launch; or goes on if a block of requests ends while the ordered core takes
    it) or goes to the ordered core, whatever the capacity."""
    lim = LIMIT[algo]
    first = -(-(lim + 64) * 4 // 3 // 64) * 64
    around = ((first - 64, MAIN, (LEAN, ORDERED)), (first, MAIN, (ORDERED,)))
    for cap, early, to in ((lim + 64, MAIN, (LEAN,)), (64, HEAVY, (ORDERED,)),
                           (lim + 64, HEAVY, (ORDERED,)), *(around if algo < 2 else ())):
        b = fragments(algo, cap + 40, more=100, seed=cap)
        res, states, status, nxt, at, free = replay(lib, b, 61440, early, cap_free=cap)
        check_refused(b, res, states, status)
        assert nxt[0] in to, f"capacity {cap}: left at request {at[0]}, {free[0]} free"


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_heavy_heaps_that_outgrow_a_small_pool(lib, algo):
    """The heavy launch, its pool outgrown by the live table while the free
    table is near a small capacity: still the ordered core."""
    for cap in (64, 320):
        b = fragments(algo, cap, more=100, seed=cap + 1)
        lives = W.Batch("lives", b.arena, b.align, b.algo, np.array([0, b.requests + 400]),
                        np.concatenate([b.req, np.full(400, 16, np.int64)]))
        pool = 8192 + 4096 if algo in (W.SEG_FIT, W.TLSF) else 8192
        res, states, status, nxt, at, free = replay(lib, lives, pool, HEAVY, cap_free=cap)
        check_refused(lives, res, states, status)
        assert nxt[0] == ORDERED, f"capacity {cap}: left at request {at[0]}, {free[0]} free"


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_largest_arena_after_the_move(lib, algo):
    """2^32 - 1 granules: blocks that end at the last granule and whole-arena
    requests on the ordered core, beside hundreds of small free blocks."""
    # (TLSF's list heads take 8 KiB of the pool)
    small, pool = (1400, 10240) if algo == W.TLSF else (500, 2048)
    b = edge_traces.fragments_then_edges(algo, (1 << 32) - 1, 64, small, 150, seed=algo)
    res, states, status, nxt, at, free = replay(lib, b, pool, HEAVY)
    assert nxt[0] == ORDERED and at[0] < 1.5 * small
    check_oracle(b, res, states, status)
