"""Traces that take a heap past its first tables and then to the arena's
edges (test helpers)."""
import numpy as np

import models
import oracle
from paper_2405_07079_amd import workloads as W


def fragments_then_edges(algo, granules, align, small, edges, seed=0):
    """One heap: `small` blocks of 1 to 4 granules, a random half of them
    freed, then `edges` requests at the arena's end -- the last free block
    taken whole, all but one granule of it, half of it; a second block taken
    from what that leaves; more than it; the whole arena; the huge blocks freed
    again, in any order (now and then, on the sequential fits and the bitmask
    allocator, all but a part of one) -- between allocations and frees of small
    blocks.  Frees name their victims by draw, so the heap is run on the oracle
    beside."""
    rng = np.random.default_rng(seed)
    o = oracle.Heap(algo, granules * align, align)
    req, live = [], []          # live: offset, size in granules

    def alloc(g):
        off = o.alloc(int(g) * align)
        req.append(int(g) * align)
        if off >= 0:
            live.append([off, int(g)])

    def free(i, keep=0):
        off, g = live[i]
        cut = -(-(keep << 31) // g) if keep else 0     # keeps floor(cut * g / 2^31) granules
        if keep and (cut * g) >> 31 == keep:
            o.free_partial(off + keep * align)
            live[i][1] = keep
        else:
            cut = 0
            o.free(off)
            live[i] = live[-1]
            live.pop()
            draw_of = i, len(live) + 1
        n = draw_of[1] if not cut else len(live)
        q = models.draw_for(i, n)
        req.append(q if not cut else -((cut << 32 | (-q - 1)) + 1))

    for g in rng.integers(1, 5, small):
        alloc(g)
    for _ in range(small // 2):
        free(int(rng.integers(len(live))))
    for _ in range(edges):
        huge = [i for i, (_, g) in enumerate(live) if g > 64]
        kind = rng.random()
        if kind < 0.25:
            alloc(rng.integers(1, 5))
        elif kind < 0.45 and len(live) > len(huge):
            i = int(rng.integers(len(live)))
            free(i)
        elif kind < 0.70 and huge:
            i = huge[int(rng.integers(len(huge)))]
            part = algo in (0, 1, 2, W.BITMAP) and rng.random() < 0.4
            free(i, int(rng.integers(1, live[i][1])) if part else 0)
        else:
            blocks = oracle.parse_state(o.state(), algo)["free"]
            rest = max((int(s) for _, s in blocks), default=0) // align
            alloc(max(1, (rest, rest - 1, rest // 2, rest + 1, granules)[int(rng.integers(5))]))
    for i in reversed(range(len(live))):                # and everything goes
        if live[i][1] > 64 or rng.random() < 0.9:
            free(i)
    alloc(granules)
    return W.Batch("edges", np.array([granules * align]), np.array([align]),
                   np.array([algo], np.int32), np.array([0, len(req)]), np.array(req, np.int64))


def without_refused(batch, res, code):
    """A batch without the requests that were refused with `code` (each changed
    nothing), and the results of the others."""
    keep = res != code
    lens = [int(keep[a:b].sum()) for a, b in zip(batch.req_off[:-1], batch.req_off[1:])]
    off = np.concatenate([[0], np.cumsum(lens)])
    return (W.Batch(batch.name, batch.arena, batch.align, batch.algo, off, batch.req[keep]),
            res[keep])
