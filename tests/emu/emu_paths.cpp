// The replay paths that start on the lean core and change core mid-trace,
// under the CPU wave emulation: the emulator of emu_replay.cpp with another
// lane program.  Test infrastructure only.
#include "emu_replay.cpp"

namespace {

struct PathJob {
  ReplayParams p;
  LeanLds lds;
  int64_t heap;
  uint64_t *bits, *nodes;  // bitmask allocator: flags, node summaries
  Ent* live;
  uint32_t kn;             // summaries kept in "LDS"
  uint64_t max_granules;
  Cold c;                  // the other allocators: the general core's tiers
  uint8_t* ord;            // and the ordered core's device slot, or null
  int done;
};
PathJob g_path;

template <int RF>
void spill_any(PathJob& j) {
  switch (j.p.algo[j.heap]) {
    case kFirstFit: lean_one_heap<kFirstFit, RF>(j.p, j.lds, j.c, j.heap, j.ord); break;
    case kNextFit: lean_one_heap<kNextFit, RF>(j.p, j.lds, j.c, j.heap, j.ord); break;
    case kBestFit: lean_one_heap<kBestFit, RF>(j.p, j.lds, j.c, j.heap, j.ord); break;
    case kSegFit: lean_one_heap<kSegFit, RF>(j.p, j.lds, j.c, j.heap, j.ord); break;
    default: lean_one_heap<kTlsf, RF>(j.p, j.lds, j.c, j.heap, j.ord); break;
  }
}

void path_main() {
  if (g_path.bits)
    bitmap_lean_heap(g_path.p, g_path.lds, g_path.bits, g_path.nodes, g_path.live, g_path.kn,
                     g_path.max_granules, g_path.heap);
  else
    spill_any<2>(g_path);
  // a finished lane keeps handing over until every lane has finished
  g_path.done++;
  for (;;) {
    const uint32_t me = emu_lane;
    if (g_path.done == 64) swapcontext(&emu_wave->lane_ctx[me], &emu_wave->main_ctx);
    const uint32_t next = (me + 1) & 63u;
    emu_lane = next;
    swapcontext(&emu_wave->lane_ctx[me], &emu_wave->lane_ctx[next]);
    emu_lane = me;
  }
}

void run_path(EmuWave& w, std::vector<std::vector<uint8_t>>& stacks) {
  for (int l = 0; l < 64; ++l) {
    getcontext(&w.lane_ctx[l]);
    w.lane_ctx[l].uc_stack.ss_sp = stacks[l].data();
    w.lane_ctx[l].uc_stack.ss_size = stacks[l].size();
    w.lane_ctx[l].uc_link = nullptr;
    makecontext(&w.lane_ctx[l], path_main, 0);
  }
  emu_lane = 0;
  g_path.done = 0;
  swapcontext(&w.main_ctx, &w.lane_ctx[0]);
}

}  // namespace

// Replay H heaps of the bitmask allocator on the table of free blocks in a
// pool of `pool` bytes, continuing on the flags (kn summaries in the pool)
// once that is too small (moved[h] = 1).  0, or 1 when a moved heap's
// summaries disagree with its flags.
extern "C" int emu_path_replay(int64_t H, const int64_t* arena, const int64_t* align,
                               const int32_t* algo, const int64_t* req_off, const int64_t* req,
                               int64_t* res, int64_t* state, const int64_t* state_off,
                               int64_t* state_len, int32_t* status, uint32_t pool, uint32_t kn,
                               uint32_t cap_live, uint8_t* moved) {
  std::memset(&g_path.p, 0, sizeof(g_path.p));
  ReplayParams& p = g_path.p;
  p.arena = arena; p.align = align; p.algo = algo; p.req_off = req_off; p.req = req;
  p.res = res; p.state = state; p.state_off = state_off; p.state_len = state_len;
  p.status = status; p.cap_live = cap_live;
  uint32_t migrated = 0;
  p.migrated = &migrated;
  std::vector<std::vector<uint8_t>> stacks(64, std::vector<uint8_t>(256 * 1024));
  EmuWave w;
  emu_wave = &w;
  int rc = 0;
  for (int64_t h = 0; h < H && rc == 0; ++h) {
    const uint64_t ag = (align[h] > 0 && arena[h] > 0) ? uint64_t(arena[h] / align[h]) : 1u;
    const uint64_t nw = (ag + 63u) / 64u, nn = (nw + 63u) / 64u;
    // poisoned, so a read of an unwritten word cannot look valid
    std::vector<uint64_t> mem(pool / 8u + 2u, 0xA5A5A5A5A5A5A5A5ull), bits(nw + 1u, mem[0]),
        nodes(nn + 1u, mem[0]);
    std::vector<Ent> live(size_t(cap_live) + 64u, mem[0]);
    g_path.lds.base = reinterpret_cast<uint8_t*>(mem.data());
    g_path.lds.bytes = pool;
    g_path.heap = h;
    g_path.bits = bits.data();
    g_path.nodes = nodes.data();
    g_path.live = live.data();
    g_path.kn = kn;
    g_path.max_granules = ag;
    const uint32_t before = migrated;
    run_path(w, stacks);
    moved[h] = migrated != before;
    if (moved[h] && status[h] == 0) {
      for (uint64_t n = 0; n < kn && n < nn; ++n) nodes[n] = mem[n];
      if (!summaries_valid(bits.data(), nodes.data(), ag)) rc = 1;
    }
  }
  emu_wave = nullptr;
  return rc;
}

// Replay H heaps on the lean core in a pool of `pool` bytes with an
// ordered-core slot for those that outgrow it (moved[h] = 1).
extern "C" int emu_spill_replay(int64_t H, const int64_t* arena, const int64_t* align,
                                const int32_t* algo, const int64_t* req_off, const int64_t* req,
                                int64_t* res, int64_t* state, const int64_t* state_off,
                                int64_t* state_len, int32_t* status, uint32_t pool,
                                uint32_t cap_free, uint32_t cap_live, uint8_t* moved) {
  std::memset(&g_path.p, 0, sizeof(g_path.p));
  ReplayParams& p = g_path.p;
  p.arena = arena; p.align = align; p.algo = algo; p.req_off = req_off; p.req = req;
  p.res = res; p.state = state; p.state_off = state_off; p.state_len = state_len;
  p.status = status; p.cap_free = cap_free; p.cap_live = cap_live;
  uint32_t migrated = 0;
  p.migrated = &migrated;
  std::vector<std::vector<uint8_t>> stacks(64, std::vector<uint8_t>(256 * 1024));
  EmuWave w;
  emu_wave = &w;
  for (int64_t h = 0; h < H; ++h) {
    std::vector<uint64_t> mem(pool / 8u + 2u, 0xA5A5A5A5A5A5A5A5ull);
    std::vector<uint64_t> slot(ord_spill_bytes(cap_free, cap_live) / 8u, mem[0]);
    g_path.lds.base = reinterpret_cast<uint8_t*>(mem.data());
    g_path.lds.bytes = pool;
    g_path.heap = h;
    g_path.bits = nullptr;
    g_path.ord = reinterpret_cast<uint8_t*>(slot.data());
    Cold& c = g_path.c;
    c.lf = nullptr; c.lst = nullptr; c.ll = nullptr;
    c.gf = reinterpret_cast<Ent*>(g_path.ord);
    c.gst = reinterpret_cast<uint32_t*>(g_path.ord + size_t(cap_free) * 8);
    c.gl = reinterpret_cast<Ent*>(g_path.ord + size_t(cap_free) * 12);
    c.kf = 0; c.kl = 0; c.cf = cap_free; c.cl = cap_live;
    const uint32_t before = migrated;
    run_path(w, stacks);
    moved[h] = migrated != before;
  }
  emu_wave = nullptr;
  return 0;
}
