"""Batches on streams of their own, side by side on one GPU: the LDS the
default plan gives each, and the results of batches in flight together."""
import numpy as np
import pytest

import oracle
from paper_2405_07079_amd import hda
from paper_2405_07079_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

QUEUES = 4                  # launches a device runs side by side
CU_LDS = 160 << 10
SMALLEST = 10 << 10         # the default pool of a full device


def say(*a):
    print(*a, flush=True)


def pool(db):
    t = hda.hda_replay_resolve(db)
    return t["lds_free"] * 16 + t["lds_live"] * 8


@pytest.mark.parametrize("heaps", (1, 100, 128, 129, 256, 257, 512, 513, 1000, 1024, 1025, 2000,
                                   2049, 4096, 20_000))
def test_default_pools_leave_room_for_other_streams(heaps):
    """Four batches of one shape fit the device's LDS at once, as they did
    with the smallest pool; few heaps still get the largest."""
    db = hda.upload(W.uniform_batch(heaps=heaps, n=1))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    waves = -(-QUEUES * heaps // cus)        # per CU, of four such batches
    p = pool(db)
    say(f"case: {heaps} heaps, {p} bytes of LDS each, {waves} waves a CU")
    assert p == SMALLEST or p * waves <= CU_LDS
    assert p == 6 * SMALLEST if waves <= 2 else p < 6 * SMALLEST


def test_batches_on_four_streams():
    """Four batches of every table algorithm at once, each on its own stream:
    results, states and statuses as the oracle's, twice in a row."""
    batches = [W.concat([W.uniform_batch(seed=10 * k + a, heaps=50 + 13 * k, n=1500, algo=a,
                                         arena=1 << 22, align=16, lo=16, hi=1 << 14)
                         for a in range(5)], "streams") for k in range(QUEUES)]
    dbs = [hda.upload(b) for b in batches]
    streams = [torch.cuda.Stream() for _ in dbs]
    torch.cuda.synchronize()
    want = [oracle.replay_batch(b, threads=8) for b in batches]
    for rep in range(2):
        say(f"case: {QUEUES} streams, {[b.heaps for b in batches]} heaps, pass {rep}")
        for db, s in zip(dbs, streams):
            hda.hda_replay(db, s)
        torch.cuda.synchronize()
        for b, db, (ores, ostates, _) in zip(batches, dbs, want):
            assert (db.status.cpu().numpy() == 0).all()
            assert np.array_equal(db.res.cpu().numpy()[:b.requests], ores)
            for h, st in enumerate(hda.states_to_host(db)):
                assert np.array_equal(st, ostates[h]), f"heap {h}"
            db.res.fill_(-7)
            db.state.fill_(-7)
        torch.cuda.synchronize()
