// The bitmask allocator's move from the table of free runs to the flags, under
// the CPU wave emulation, with the cross-lane steps it took.  Test
// infrastructure only.
#include "emu_paths.cpp"

// One heap as in emu_path_replay; *steps receives the rounds of cross-lane
// steps of the whole replay.  0, or 1 when the summaries disagree with the
// flags of a moved heap.
extern "C" int emu_take_replay(int64_t arena, int64_t align, int64_t n, const int64_t* req,
                               int64_t* res, int64_t* state, int64_t state_cap,
                               int64_t* state_len, int32_t* status, uint32_t pool, uint32_t kn,
                               uint32_t cap_live, uint32_t* moved, uint64_t* steps) {
  std::memset(&g_path.p, 0, sizeof(g_path.p));
  ReplayParams& p = g_path.p;
  const int32_t algo = kBitmap;
  const int64_t off[2] = {0, n}, soff[2] = {0, state_cap};
  p.arena = &arena; p.align = &align; p.algo = &algo; p.req_off = off; p.req = req;
  p.res = res; p.state = state; p.state_off = soff; p.state_len = state_len;
  p.status = status; p.cap_live = cap_live;
  *moved = 0;
  p.migrated = moved;
  std::vector<std::vector<uint8_t>> stacks(64, std::vector<uint8_t>(256 * 1024));
  EmuWave w;
  emu_wave = &w;
  const uint64_t ag = uint64_t(arena / align), nw = (ag + 63u) / 64u, nn = (nw + 63u) / 64u;
  std::vector<uint64_t> mem(pool / 8u + 2u, 0xA5A5A5A5A5A5A5A5ull), bits(nw + 1u, mem[0]),
      nodes(nn + 1u, mem[0]);
  std::vector<Ent> live(size_t(cap_live) + 64u, mem[0]);
  g_path.lds.base = reinterpret_cast<uint8_t*>(mem.data());
  g_path.lds.bytes = pool;
  g_path.heap = 0;
  g_path.bits = bits.data();
  g_path.nodes = nodes.data();
  g_path.live = live.data();
  g_path.kn = kn;
  g_path.max_granules = ag;
  run_path(w, stacks);
  *steps = w.syncs;
  emu_wave = nullptr;
  if (*moved == 0 || *status != 0) return 0;
  for (uint64_t i = 0; i < kn && i < nn; ++i) nodes[i] = mem[i];
  return bits[nw] == 0xA5A5A5A5A5A5A5A5ull && nodes[nn] == bits[nw] &&
                 summaries_valid(bits.data(), nodes.data(), ag)
             ? 0
             : 1;
}
