"""Which tunings a replay takes and refuses, whatever the number of heaps (host
side: nothing is launched)."""
import pytest

from paper_2405_07079_amd import hda
from paper_2405_07079_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def takes(db, **kw):
    db.tuning = hda.tuning(**kw)
    try:
        hda.hda_replay_workspace(db)
        return True
    except hda.HdaError as e:
        assert e.code == hda.HDA_E_INVAL
        return False


@pytest.mark.parametrize("heaps", (1, 1024, 1025, 2048, 2049, 5000))
def test_lds_sizes_are_judged_alike_for_every_batch(heaps):
    """LDS sizes asked for without heaps_per_group: taken up to what four waves
    of a workgroup can hold of the 160 KiB, at every batch size."""
    db = hda.upload(W.uniform_batch(heaps=heaps, n=1))
    print("case:", heaps, "heaps", flush=True)
    assert takes(db)
    assert takes(db, lds_free=2048) and takes(db, lds_live=4096)      # 40 / 34 KiB a wave
    assert not takes(db, lds_free=4096) and not takes(db, lds_live=8192)
    assert not takes(db, lds_free=2112, lds_live=1024)                # 164 KiB for four
    assert takes(db, lds_free=4096, heaps_per_group=1)
    assert not takes(db, lds_free=4096, heaps_per_group=4)
    # what a plan resolves to is itself a tuning that is taken
    db.tuning = hda.tuning()
    r = hda.hda_replay_resolve(db)
    assert takes(db, **{k: r[k] for k in hda.TUNING_FIELDS})
