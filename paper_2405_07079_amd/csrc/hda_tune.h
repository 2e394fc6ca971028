// The autotuner's candidates (host side).
#pragma once
#include <stdint.h>

#include <vector>

#include "hda.h"

namespace hda {

// Tunings to time for the lean path: heaps per workgroup by LDS residency,
// and the default plan of the whole batch (`plan`, as resolved), which gives
// few heaps larger pools than any of the others: what the autotuner returns
// is then never slower than not tuning, as far as its trial shows.  The other
// fields are `base`'s.
inline std::vector<hda_tuning> lean_candidates(const hda_tuning& base, const hda_tuning& plan) {
  std::vector<hda_tuning> out;
  const auto add = [&](int32_t waves, int32_t lds_free, int32_t lds_live) {
    for (const hda_tuning& t : out)
      if (t.heaps_per_group == waves && t.lds_free == lds_free && t.lds_live == lds_live) return;
    hda_tuning t = base;
    t.heaps_per_group = waves;
    t.reg_free = t.reg_free < 0 ? 0 : t.reg_free;
    t.reg_live = 0;
    t.lds_free = lds_free;
    t.lds_live = lds_live;
    t.groups = 0;
    t.heavy_heaps = 0;
    t.heavy_kib = 0;
    out.push_back(t);
  };
  const int32_t lds_pairs[][2] = {{64, 512}, {128, 1024}, {256, 2048}, {512, 4096}};
  for (int32_t waves : {1, 2, 4, 8, 16})
    for (const auto& kv : lds_pairs) add(waves, kv[0], kv[1]);
  add(plan.heaps_per_group, plan.lds_free, plan.lds_live);
  return out;
}

}  // namespace hda
