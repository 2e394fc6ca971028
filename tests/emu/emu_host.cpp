// The host code of the call-by-call heaps (hda_heap.hip) on the CPU, with the
// HIP runtime's stand-in of tests/emu/host.  Compiled beside a copy of the
// sources in which hda_wave.h is emu_wave.h.  Test infrastructure only.
#include <ucontext.h>

#include <cstdint>
#include <mutex>
#include <vector>

#include "emu_wave.h"
#include "hda_heap.hip"

namespace hda {
EmuWave* emu_wave = nullptr;
uint32_t emu_lane = 0;
}  // namespace hda

void (*emu_on_host_free)() = nullptr;
int emu_host_pages = 0;
int emu_stream_waits = 0;

extern "C" void emu_set_on_host_free(void (*f)()) { emu_on_host_free = f; }
extern "C" int emu_pages() { return emu_host_pages; }
extern "C" int emu_waits() { return emu_stream_waits; }

namespace {

const std::function<void()>* g_body;
int g_done;

void lane_main() {
  (*g_body)();
  // a finished lane keeps handing over until every lane has finished
  g_done++;
  for (;;) {
    const uint32_t me = hda::emu_lane;
    if (g_done == 64) swapcontext(&hda::emu_wave->lane_ctx[me], &hda::emu_wave->main_ctx);
    const uint32_t next = (me + 1) & 63u;
    hda::emu_lane = next;
    swapcontext(&hda::emu_wave->lane_ctx[me], &hda::emu_wave->lane_ctx[next]);
    hda::emu_lane = me;
  }
}

}  // namespace

void emu_run_wave(const std::function<void()>& f) {
  static std::mutex mu;  // one wave at a time
  static std::vector<std::vector<uint8_t>> stacks(64, std::vector<uint8_t>(256 * 1024));
  static hda::EmuWave w;
  std::lock_guard<std::mutex> g(mu);
  hda::emu_wave = &w;
  g_body = &f;
  g_done = 0;
  for (int l = 0; l < 64; ++l) {
    getcontext(&w.lane_ctx[l]);
    w.lane_ctx[l].uc_stack.ss_sp = stacks[l].data();
    w.lane_ctx[l].uc_stack.ss_size = stacks[l].size();
    w.lane_ctx[l].uc_link = nullptr;
    makecontext(&w.lane_ctx[l], lane_main, 0);
  }
  hda::emu_lane = 0;
  swapcontext(&w.main_ctx, &w.lane_ctx[0]);
}
