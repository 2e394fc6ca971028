"""The work this framework is used for, as cases that can be timed.

Every case is a dict of plain values; `family` says which of the public entry
points it goes through and how its inputs are made:

* ``batch``  -- many independent heaps with equal or ragged traces, replayed by
  ``hda_replay`` (also captured as a graph, or through ``hda_replay_static``)
  or, for the bitmask allocator, by ``hda_bitmap_replay``;
* ``uneven`` -- heaps of very different arenas and trace lengths, all four
  basic allocators mixed, with the default tuning or with the longest heaps on
  the ordered core;
* ``large``  -- one heap over a very large arena, on the ordered core;
* ``calls``  -- one heap driven call by call.

The service (``Server``) is a kernel that runs until it is stopped and is
measured by its own open-loop load generator, not by timed passes; it runs the
same allocator code as the call-by-call heaps.

Results are byte offsets, states and status codes: whole numbers, equal bit
for bit on every path.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2405_07079_amd import hda
from paper_2405_07079_amd import workloads as W

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
MIXED = -1            # heap h runs algorithm h mod 5
META_FREE, META_LIVE = 4096, 8192


def _batch(name, **kw):
    c = dict(name=name, family="batch", entry="replay", algo=W.BEST_FIT, heaps=4096,
             arena=16 * MiB, align=64, n=100_000, p_alloc=0.55, lo=64, hi=1 * MiB,
             partial=0.0, ragged=False)
    c.update(kw)
    return c


def listed():
    return [
        # a program that allocates and frees device memory one call at a time
        # (blocks of 1 KiB to 16 MiB from a 4 GiB heap of 4 KiB granules, the
        # setting of the paper's experiment): launch and wait per call
        dict(name="heap_calls_seg_fit", family="calls", algo=W.SEG_FIT, arena=4 * GiB,
             align=4 * KiB, warm=2500, calls=16, lo=1 * KiB, hi=16 * MiB, partial=False),
        # the smallest replay: one small heap, one dependent chain of requests
        _batch("one_heap_first_fit", algo=W.FIRST_FIT, heaps=1, arena=64 * KiB, align=16,
               n=10_000, p_alloc=0.6, lo=16, hi=4 * KiB),
        # a handful of short ragged traces, every allocator, as a captured
        # graph that a program launches again and again
        _batch("short_mixed_graph", algo=MIXED, heaps=48, n=500, ragged=True, entry="graph"),
        # the benchmark's two replays: a full device of equal heaps
        _batch("heaps_4096_best_fit", algo=W.BEST_FIT),
        _batch("heaps_4096_seg_fit", algo=W.SEG_FIT),
        # the same batch (shorter traces) on two-level segregated fit and on
        # the bitmask allocator, and on best fit with partial frees
        _batch("heaps_4096_tlsf", algo=W.TLSF, n=40_000),
        _batch("heaps_4096_bitmask", algo=W.BITMAP, n=40_000),
        _batch("heaps_4096_partial_frees", algo=W.BEST_FIT, n=40_000, partial=0.02),
        # fewer heaps than the device holds, ragged, with small blocks: the
        # tables grow to thousands of entries
        _batch("ragged_small_blocks_next_fit", algo=W.NEXT_FIT, heaps=1000, align=16, n=30_000,
               lo=16, hi=64 * KiB, ragged=True),
        # arenas of 1 MiB to 1 GiB and Pareto trace lengths, four allocators
        # mixed: with the default tuning, and with the tuning the autotuner
        # picks for such a batch
        dict(name="uneven_default", family="uneven", heaps=16_384, len_hi=200_000, heavy=0),
        dict(name="uneven_heavy", family="uneven", heaps=16_384, len_hi=200_000, heavy=128),
        # one 256 GiB heap of 4 KiB granules on segregated fit, the first
        # million requests of such a trace
        dict(name="large_256GiB_seg_fit", family="large", algo=W.SEG_FIT, arena=256 * GiB,
             n=1_000_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: batches of 1 to 4,096 heaps and 100
    to 100,000 requests each over arenas of 64 KiB to 1 GiB, blocks up to 1/16
    to 1/256 of the arena, every allocator; uneven batches; large heaps; call
    by call heaps."""
    family = rng.choice(["batch", "batch", "batch", "batch", "uneven", "large", "calls"])
    if family == "calls":
        align = rng.choice([64, 512, 4096])
        arena = _log(rng, 256 * KiB, 64 * GiB) // align * align
        algo = rng.randrange(5)
        return dict(family="calls", algo=algo, arena=arena, align=align,
                    warm=_log(rng, 10, 5000), calls=_log(rng, 1, 64), lo=align,
                    hi=max(2 * align, arena // rng.choice([64, 256])),
                    partial=algo <= W.BEST_FIT and rng.random() < 0.5)
    if family == "uneven":
        return dict(family="uneven", heaps=_log(rng, 256, 16_384),
                    len_hi=_log(rng, 10_000, 200_000), heavy=rng.choice([0, 16, 64, 128]))
    if family == "large":
        return dict(family="large", algo=rng.randrange(5), arena=1 << rng.randint(32, 38),
                    n=_log(rng, 20_000, 800_000))
    algo = rng.choice([0, 1, 2, 3, 4, W.BITMAP, MIXED])
    align = rng.choice([16, 32, 64, 512])
    # the bitmask allocator's arenas end at 2^20 granules here
    arena = _log(rng, 64 * KiB, min(1 * GiB, align << 20 if algo == W.BITMAP else 1 * GiB))
    arena = max(arena // align * align, 1024 * align)
    k = rng.randint(4, 8)
    heaps = _log(rng, 1, 4096)
    entry = rng.choice(["replay", "replay", "graph", "static"])
    if algo == W.BITMAP or (entry == "static" and heaps > 512):  # static scratch is bounded
        entry = "replay"
    return dict(family="batch", entry=entry, algo=algo, heaps=heaps, arena=arena, align=align,
                n=_log(rng, 100, 100_000 >> max(0, k - 6)), p_alloc=rng.choice([0.5, 0.55, 0.6]),
                lo=align, hi=max(2 * align, arena >> k),
                partial=rng.choice([0.0, 0.0, 0.02, 0.1]), ragged=rng.random() < 0.5)


# ---- inputs, drawn on the GPU ----

def _stream(g, n, sizes, p_alloc, partial):
    """n requests: allocate sizes[i] with probability p_alloc, else free a
    uniform live block (a 32-bit draw, and a cut for a partial free)."""
    dev = sizes.device
    u = torch.randint(0, 1 << 32, (n,), generator=g, device=dev, dtype=torch.int64)
    if partial > 0.0:
        cut = torch.randint(1, 1 << 31, (n,), generator=g, device=dev, dtype=torch.int64)
        part = torch.rand(n, generator=g, device=dev) < partial
        u |= torch.where(part, cut, torch.zeros_like(cut)) << 32
    dec = torch.rand(n, generator=g, device=dev)
    return torch.where(dec < p_alloc, sizes, -(u + 1))


def _log_uniform(g, n, lo, hi, dev):
    """floor(lo (hi / lo)^u) clamped to [lo, hi]; hi a number or one per request."""
    v = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
    hi = torch.as_tensor(hi, dtype=torch.float64, device=dev)
    v.mul_(torch.log(hi / lo)).exp_().mul_(lo).floor_()
    return torch.minimum(v.clamp_(min=lo), hi).to(torch.int64)


def _device_batch(arena, align, algo, lens, req, tuning=(), meta_free=META_FREE,
                  meta_live=META_LIVE):
    """A DeviceBatch over requests already on the GPU, with outputs, states
    and the library's workspace; longest traces first."""
    dev = req.device
    H = len(lens)
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a, dt)).to(dev)  # noqa: E731
    blocks = np.where(algo == W.BITMAP, np.minimum(2 * lens + 1, 2 * meta_live + 1),
                      np.minimum(lens + 1, meta_free + meta_live))
    off, soff = np.zeros(H + 1, np.int64), np.zeros(H + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    np.cumsum(hda.state_words(algo, blocks), out=soff[1:])
    # the slots are larger than the states: what no replay writes stays zero
    db = hda.DeviceBatch(H, t(arena, np.int64), t(align, np.int64), t(algo, np.int32),
                         t(off, np.int64), req, torch.empty_like(req),
                         t(np.argsort(-lens, kind="stable"), np.int32),
                         torch.zeros(int(soff[-1]), dtype=torch.int64, device=dev),
                         t(soff, np.int64), torch.zeros(H, dtype=torch.int64, device=dev),
                         torch.zeros(H, dtype=torch.int32, device=dev), meta_free, meta_live)
    return hda.retune(db, tuning or hda.tuning())


# Arenas and trace lengths are part of the case (seeds of their own); the
# requests come from the seed that prepare() is given.
def _prepare_batch(c, g, rng, dev):
    H, n, align = c["heaps"], c["n"], c["align"]
    lens = np.full(H, n, np.int64)
    arena = np.full(H, c["arena"], np.int64)
    if c["ragged"]:
        rng = np.random.Generator(np.random.PCG64(2))
        lens -= rng.integers(0, n // 2 + 1, H)
        arena = np.maximum(arena - rng.integers(0, c["arena"] // 4, H) // align * align, align)
    algo = np.full(H, c["algo"], np.int32) if c["algo"] != MIXED else \
        (np.arange(H) % 5).astype(np.int32)
    N = int(lens.sum())
    req = _stream(g, N, _log_uniform(g, N, c["lo"], c["hi"], dev), c["p_alloc"], c["partial"])
    return _device_batch(arena, np.full(H, align, np.int64), algo, lens, req)


def _prepare_uneven(c, g, rng, dev):
    arena, lens, algo = W.uneven_params(3, c["heaps"], len_hi=c["len_hi"])
    N = int(lens.sum())
    hi = torch.repeat_interleave(torch.from_numpy(arena).to(dev),
                                 torch.from_numpy(lens).to(dev)).to(torch.float64) / 64
    req = _stream(g, N, _log_uniform(g, N, 32, hi, dev), 0.55, 0.0)
    tuning = hda.tuning(heaps_per_group=4, lds_free=512, lds_live=4096, heavy_heaps=c["heavy"],
                        heavy_kib=64) if c["heavy"] else hda.tuning()
    return _device_batch(arena, np.full(c["heaps"], 32, np.int64), algo, lens, req, tuning)


def _prepare_large(c, g, rng, dev):
    n = c["n"]
    # class k = 12..26 with probability 2^-(k - 11), a size uniform over the
    # multiples of 4 KiB in (2^(k-1), 2^k]
    k = 12 + torch.clamp((-torch.log2(1 - torch.rand(n, generator=g, device=dev,
                                                     dtype=torch.float64))).floor(), max=14)
    k = k.to(torch.int64)
    choices = torch.clamp((1 << (k - 1)) // 4096, min=1)
    i = (torch.rand(n, generator=g, device=dev, dtype=torch.float64) * choices).to(torch.int64)
    req = _stream(g, n, (1 << k) - 4096 * i, 0.5, 0.0)
    one = lambda x, dt: np.array([x], dt)  # noqa: E731
    return _device_batch(one(c["arena"], np.int64), one(4096, np.int64),
                         one(c["algo"], np.int32), one(n, np.int64), req,
                         hda.tuning(heavy_heaps=1, heavy_kib=158), 4096, 16_384)


def _prepare_calls(c, g, rng, dev):
    """A heap in mid-life (the state that `warm` requests leave) and the sizes
    of the next calls."""
    w = c["warm"]
    req = _stream(g, w, _log_uniform(g, w, c["lo"], c["hi"], dev), 0.55, 0.0)
    one = lambda x, dt: np.array([x], dt)  # noqa: E731
    db = _device_batch(one(c["arena"], np.int64), one(c["align"], np.int64),
                       one(c["algo"], np.int32), one(w, np.int64), req)
    hda.hda_replay(db)
    torch.cuda.synchronize()
    heap = hda.Heap(c["arena"], c["align"], c["algo"])
    if heap.load(hda.states_to_host(db)[0]) != hda.HDA_OK:
        raise RuntimeError("the heap did not take its state")
    sizes = np.exp(rng.uniform(math.log(c["lo"]), math.log(c["hi"]), c["calls"]))
    least = c["align"] + 1 if c["partial"] else 1   # a partial free keeps one granule
    return dict(heap=heap, sizes=[max(int(s), least) for s in sizes])


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    make = dict(batch=_prepare_batch, uneven=_prepare_uneven, large=_prepare_large,
                calls=_prepare_calls)[case["family"]]
    state = make(case, g, rng, dev)
    if case["family"] == "calls":
        state["case"] = case
        return state
    state = dict(case=case, db=state)
    if case.get("entry") == "graph":
        state["graph"] = hda.ReplayGraph(state["db"])
    return state


def _run_calls(state):
    """Allocate every size, then free in the reverse order (partial: the tail
    of each block first), which leaves the heap as it was.  A code of 0 stands
    where nothing was allocated."""
    heap, align = state["heap"], state["case"]["align"]
    out = [heap.alloc(s) for s in state["sizes"]]
    codes = []
    for off in reversed(out):
        if state["case"]["partial"]:
            codes.append(heap.free_partial(off + align) if off >= 0 else 0)
        codes.append(heap.free(off) if off >= 0 else 0)
    return np.array(out + codes, np.int64)


def run(state):
    case = state["case"]
    if case["family"] == "calls":
        return _run_calls(state)
    db = state["db"]
    if case.get("algo") == W.BITMAP:
        hda.hda_bitmap_replay(db, case["arena"] // case["align"])
    elif "graph" in state:
        state["graph"].launch()
    elif case.get("entry") == "static":
        hda.hda_replay_static(db)
    else:
        hda.hda_replay(db)
    return dict(res=db.res, state=db.state, state_len=db.state_len, status=db.status)


def work(case):
    """Each request is read once and its result written once, 8 bytes each
    (uneven batches: about 2,800 requests per heap at the longest cut); a call
    reads and writes the entries of about two blocks."""
    if case["family"] == "calls":
        return dict(bytes=64 * 2 * case["calls"], flops=0)
    if case["family"] == "uneven":
        mean = 1000 * (3 - 2 * math.sqrt(1000 / case["len_hi"]))  # of the clipped Pareto lengths
        return dict(bytes=16 * int(case["heaps"] * mean), flops=0)
    if case["family"] == "large":
        return dict(bytes=16 * case["n"], flops=0)
    return dict(bytes=int(16 * case["heaps"] * case["n"] * (0.75 if case["ragged"] else 1.0)),
                flops=0)
