"""Replays whose tables outgrow the lean pool, on the GPU against the oracle
(results, final states): the ordered-core continuation, the general core in a
workspace without its slots, and the pool sizes of small batches."""
import numpy as np
import pytest

import oracle
from paper_2405_07079_amd import hda
from paper_2405_07079_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True)


def check(batch, db):
    torch.cuda.synchronize()
    res, status = db.res.cpu().numpy()[:batch.requests], db.status.cpu().numpy()
    states = hda.states_to_host(db)
    ores, ostates, _ = oracle.replay_batch(batch, threads=8)
    assert (status == 0).all()
    assert np.array_equal(res, ores)
    for h in range(batch.heaps):
        assert np.array_equal(states[h], ostates[h]), f"heap {h}"


def small_blocks(heaps, n, algo, **kw):
    return W.uniform_batch(seed=17, heaps=heaps, arena=1 << 22, align=16, n=n, p_alloc=0.6,
                           lo=16, hi=8192, algo=algo, p_partial=0.1, name="small", **kw)


# heaps in flight per CU and the pool they get: 60, 40, 20 and 10 KiB
@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
@pytest.mark.parametrize("heaps,n", ((3, 20_000), (700, 6000), (1500, 6000), (2400, 6000)))
def test_tables_outgrow_the_pool(algo, heaps, n):
    b = small_blocks(heaps, n, algo)
    say(f"case: {heaps} heaps of small blocks, {n} requests, algo {algo}")
    db = hda.upload(b, meta_live=16_384)
    hda.hda_replay(db)
    check(b, db)


@pytest.mark.parametrize("entry", ("workspace", "static", "graph"))
def test_workspace_without_ordered_slots(entry):
    """A workspace that holds the general core's slots but not the ordered
    core's (as the static scratch does for 400 heaps) is still taken."""
    b = W.concat([small_blocks(80, 4000, a) for a in range(5)], "mixed")
    db = hda.upload(b)
    # 16 lists / counters, then 12 bytes per free and 8 per live entry and wave
    waves = (b.heaps + 3) // 4 * 4
    small = waves * (4096 * 12 + 8192 * 8) + 8 * b.heaps + 65536
    need = hda.hda_replay_workspace(db)
    assert small < need
    say(f"case: {b.heaps} heaps, {entry}, workspace {small} of {need} bytes")
    if entry == "static":
        assert need > hda.STATIC_SCRATCH_BYTES >= small
        hda.hda_replay_static(db)
    else:
        db.workspace = torch.empty(small, dtype=torch.uint8, device="cuda")
        if entry == "graph":
            g = hda.ReplayGraph(db)
            for _ in range(3):
                db.res.fill_(77)
                g.launch()
                check(b, db)
            g.close()
        else:
            hda.hda_replay(db)
    check(b, db)
    db.workspace = torch.empty(4096, dtype=torch.uint8, device="cuda")
    with pytest.raises(hda.HdaError) as e:
        hda.hda_replay(db)
    assert e.value.code == hda.HDA_E_RANGE


@pytest.mark.parametrize("algo", (0, 1, 2, 3, 4))
def test_ordered_launch_alone(algo):
    """Every heap on the ordered core: no other launch; LDS pools whose live
    part is not a whole number of chunks."""
    b = W.concat([W.uniform_batch(seed=4, heaps=2, n=6000, algo=algo),
                  small_blocks(2, 9000, algo)])
    for kib in (16, 17, 33):
        say(f"case: 4 heaps, all on the ordered core, {kib} KiB, algo {algo}")
        db = hda.upload(b, tuning=hda.tuning(heavy_heaps=b.heaps, heavy_kib=kib))
        hda.hda_replay(db)
        check(b, db)


@pytest.mark.parametrize("threads", (1, 6))
def test_heap_calls_from_threads(threads):
    """Call-by-call heaps side by side (more than a page of result words), each
    driven by one of several threads, results and states as the oracle's;
    results of every kind: offsets, -1, refusals, dumps between calls."""
    import threading
    A, g, n = 1 << 20, 64, 40
    heaps = [(hda.Heap(A, g, k % 5), oracle.Heap(k % 5, A, g)) for k in range(70)]
    say(f"case: {len(heaps)} heaps, {threads} threads, {n} rounds")
    errors = []

    def drive(t):
        try:
            for k in range(t, len(heaps), threads):
                h, o = heaps[k]
                rng = np.random.default_rng(k)
                live = []
                for i in range(n):
                    size = int(rng.integers(0, A // 8)) if i % 9 else 2 * A
                    off = h.alloc(size)
                    assert off == o.alloc(size)
                    if off >= 0:
                        live.append(off)
                    if live and i % 3 == 0:
                        x = live.pop(int(rng.integers(len(live))))
                        assert h.free(x) == o.free(x) == 0
                        assert h.free(x) == hda.HDA_E_BADFREE
                assert np.array_equal(h.state(), o.state())
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=drive, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors[0]
    for h, _ in heaps:
        h.close()
