// One call on a device-resident heap under the CPU wave emulation, looking at
// the heap's memory at the moment the call's result is published.  Test
// infrastructure only.
#include <ucontext.h>

#include <cstdint>
#include <cstring>
#include <vector>

#include "emu_wave.h"

namespace {
void emu_publish(int64_t* word, int64_t r, bool release);
}
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_store(p, v, order, scope) emu_publish(p, v, (order) == __ATOMIC_RELEASE)

#include "hda_core.h"
#include "hda_heap_dev.h"

namespace hda {
EmuWave* emu_wave = nullptr;
uint32_t emu_lane = 0;
}  // namespace hda

using namespace hda;

namespace {

struct CallJob {
  HeapHdr* hd;
  int op;
  int64_t arg;
  int64_t* dump;
  int64_t cap;
  int64_t* word;
  std::vector<uint8_t>* seen;  // the heap's bytes as published
  bool released;
  int done;
};
CallJob g_call;

void emu_publish(int64_t* word, int64_t r, bool release) {
  const uint8_t* b = reinterpret_cast<const uint8_t*>(g_call.hd);
  g_call.seen->assign(b, b + heap_bytes(g_call.hd->cf, g_call.hd->cl));
  g_call.released = release;
  *word = r;
}

void call_main() {
  CallJob& j = g_call;
  switch (j.hd->algo) {
    case kFirstFit: heap_call_t<kFirstFit>(j.hd, j.op, j.arg, j.dump, j.cap, j.word); break;
    case kNextFit: heap_call_t<kNextFit>(j.hd, j.op, j.arg, j.dump, j.cap, j.word); break;
    case kBestFit: heap_call_t<kBestFit>(j.hd, j.op, j.arg, j.dump, j.cap, j.word); break;
    case kSegFit: heap_call_t<kSegFit>(j.hd, j.op, j.arg, j.dump, j.cap, j.word); break;
    default: heap_call_t<kTlsf>(j.hd, j.op, j.arg, j.dump, j.cap, j.word); break;
  }
  // a finished lane keeps handing over until every lane has finished
  j.done++;
  for (;;) {
    const uint32_t me = emu_lane;
    if (j.done == 64) swapcontext(&emu_wave->lane_ctx[me], &emu_wave->main_ctx);
    const uint32_t next = (me + 1) & 63u;
    emu_lane = next;
    swapcontext(&emu_wave->lane_ctx[me], &emu_wave->lane_ctx[next]);
    emu_lane = me;
  }
}

}  // namespace

// Run n calls (op[i], arg[i]) on a new heap of `cap` entries per table.
// res[i] is the published result; early[i] = 1 if it was published before the
// heap's memory was as the call left it, or not as a release.
extern "C" int emu_heap_calls(int algo, int64_t arena, int64_t align, uint32_t cap, int64_t n,
                              const int32_t* op, const int64_t* arg, int64_t* res,
                              uint8_t* early) {
  std::vector<uint64_t> mem(heap_bytes(cap, cap) / 8u + 1u, 0xA5A5A5A5A5A5A5A5ull);
  HeapHdr* hd = reinterpret_cast<HeapHdr*>(mem.data());
  std::memset(hd, 0, sizeof(*hd));
  hd->algo = algo;
  hd->arena = arena;
  hd->shift = (uint32_t)__builtin_ctzll((uint64_t)align);
  hd->ag = (uint32_t)(arena / align);
  hd->cf = cap;
  hd->cl = cap;
  std::vector<std::vector<uint8_t>> stacks(64, std::vector<uint8_t>(256 * 1024));
  std::vector<int64_t> dump(8192);
  std::vector<uint8_t> seen;
  EmuWave w;
  emu_wave = &w;
  for (int64_t i = -1; i < n; ++i) {  // (-1: the heap's first call)
    int64_t word = INT64_MIN;
    g_call = CallJob{hd, i < 0 ? (int)kOpInit : op[i], i < 0 ? 0 : arg[i], dump.data(),
                     (int64_t)dump.size(), &word, &seen, false, 0};
    for (int l = 0; l < 64; ++l) {
      getcontext(&w.lane_ctx[l]);
      w.lane_ctx[l].uc_stack.ss_sp = stacks[l].data();
      w.lane_ctx[l].uc_stack.ss_size = stacks[l].size();
      w.lane_ctx[l].uc_link = nullptr;
      makecontext(&w.lane_ctx[l], call_main, 0);
    }
    emu_lane = 0;
    swapcontext(&w.main_ctx, &w.lane_ctx[0]);
    if (i < 0) continue;
    res[i] = word;
    early[i] = !g_call.released || seen.size() != heap_bytes(cap, cap) ||
               std::memcmp(seen.data(), hd, seen.size()) != 0;
  }
  emu_wave = nullptr;
  return 0;
}
