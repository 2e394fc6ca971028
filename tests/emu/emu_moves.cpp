// Where a heap goes when it leaves the lean core, under the CPU wave
// emulation: the parts of the lean path run as the GPU kernels run them
// (lean_start, then ord_continue or general_continue).  Test infrastructure
// only.
#include "emu_paths.cpp"

namespace {

int g_early;
LeanExit g_exit;

template <int ALGO>
void move_heap(PathJob& j) {
  const LeanExit x = lean_start<ALGO, 2>(j.p, j.lds, j.c, j.heap, j.ord);
  if (lane_id() == 0) g_exit = x;
  if (x.next == LeanExit::kOrdered) ord_continue<ALGO>(j.p, j.lds, j.ord, j.heap, x);
  if (x.next == LeanExit::kGeneral) general_continue<ALGO>(j.p, j.c, j.heap, x);
}

void move_main() {
  switch (g_path.p.algo[g_path.heap]) {
    case kFirstFit: move_heap<kFirstFit>(g_path); break;
    case kNextFit: move_heap<kNextFit>(g_path); break;
    case kBestFit: move_heap<kBestFit>(g_path); break;
    case kSegFit: move_heap<kSegFit>(g_path); break;
    default: move_heap<kTlsf>(g_path); break;
  }
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

}  // namespace

// Replay H heaps on the lean core in a pool of `pool` bytes with an
// ordered-core slot; `early` is ReplayParams::lean_early.  next[h]: 0 the heap
// ended on the lean core, 1 it went on to the ordered core, 2 to the general
// core; at[h] and free[h]: the request it left at and its free blocks then.
extern "C" int emu_move_replay(int64_t H, const int64_t* arena, const int64_t* align,
                               const int32_t* algo, const int64_t* req_off, const int64_t* req,
                               int64_t* res, int64_t* state, const int64_t* state_off,
                               int64_t* state_len, int32_t* status, uint32_t pool, int early,
                               uint32_t cap_free, uint32_t cap_live, int32_t* next, int64_t* at,
                               int64_t* free_blocks) {
  std::memset(&g_path.p, 0, sizeof(g_path.p));
  ReplayParams& p = g_path.p;
  p.arena = arena; p.align = align; p.algo = algo; p.req_off = req_off; p.req = req;
  p.res = res; p.state = state; p.state_off = state_off; p.state_len = state_len;
  p.status = status; p.cap_free = cap_free; p.cap_live = cap_live;
  p.lean_early = early;
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
    for (int l = 0; l < 64; ++l) {
      getcontext(&w.lane_ctx[l]);
      w.lane_ctx[l].uc_stack.ss_sp = stacks[l].data();
      w.lane_ctx[l].uc_stack.ss_size = stacks[l].size();
      w.lane_ctx[l].uc_link = nullptr;
      makecontext(&w.lane_ctx[l], move_main, 0);
    }
    emu_lane = 0;
    g_path.done = 0;
    swapcontext(&w.main_ctx, &w.lane_ctx[0]);
    next[h] = g_exit.next;
    at[h] = g_exit.pos - req_off[h];
    free_blocks[h] = g_exit.F;
  }
  emu_wave = nullptr;
  return 0;
}
