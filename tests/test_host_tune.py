"""The autotuner's candidates, compiled for the host alone."""
import ctypes
import os
import subprocess
import tempfile

import pytest

import emu
from paper_2405_07079_amd import hda

SRC = r"""
#include "hda_tune.h"
extern "C" int candidates(const hda_tuning* base, const hda_tuning* plan, hda_tuning* out, int cap) {
  const std::vector<hda_tuning> c = hda::lean_candidates(*base, *plan);
  for (int i = 0; i < (int)c.size() && i < cap; ++i) out[i] = c[(size_t)i];
  return (int)c.size();
}
"""


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "tune.cpp"), os.path.join(d, "tune.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", emu.CSRC,
                               "-I", os.path.join(emu.ROOT, "include"), src, "-o", so])
        yield ctypes.CDLL(so)


def candidates(lib, base, plan):
    out = (hda.hda_tuning * 64)()
    n = lib.candidates(ctypes.byref(hda.hda_tuning(*base)), ctypes.byref(hda.hda_tuning(*plan)),
                       out, 64)
    return [tuple(getattr(t, f) for f in hda.TUNING_FIELDS) for t in out[:n]]


# the default plans of few heaps (60, 40 and 20 KiB pools) and of a full device
@pytest.mark.parametrize("plan", ((1, 768, 6144), (1, 512, 4096), (1, 256, 2048), (4, 128, 1024)))
def test_the_default_plan_is_a_candidate(lib, plan):
    resolved = hda.tuning(heaps_per_group=plan[0], reg_free=2, reg_live=-1, lds_free=plan[1],
                          lds_live=plan[2], groups=100)
    got = candidates(lib, hda.tuning(reg_free=4, groups=7, heavy_heaps=3, heavy_kib=64), resolved)
    assert hda.tuning(heaps_per_group=plan[0], reg_free=4, lds_free=plan[1],
                      lds_live=plan[2]) in got
    assert len(set(got)) == len(got)             # timed once each
    for waves in (1, 2, 4, 8, 16):
        for f, l in ((64, 512), (128, 1024), (256, 2048), (512, 4096)):
            assert hda.tuning(heaps_per_group=waves, reg_free=4, lds_free=f, lds_live=l) in got
    # the general path is not a candidate: its tunings are timed on the lean one
    assert {t[1] for t in candidates(lib, hda.tuning(reg_free=-1), resolved)} == {0}
