// One heap's replay by one wavefront: validate its parameters, initialise
// the tables (Alg. 6), run its requests in order and write results and the
// canonical state.  Shared by the persistent and the per-heap launches.
#pragma once
#include <stdint.h>

#include "hda_bitmap.h"
#include "hda_core.h"
#include "hda_lean.h"
#include "hda_ordered.h"

namespace hda {

constexpr int kBitmapRF = 2;  // free-table chunks in registers (bitmask allocator)

struct ReplayParams {
  const int64_t* arena;
  const int64_t* align;
  const int32_t* algo;
  const int64_t* req_off;
  const int64_t* req;
  int64_t* res;
  const int32_t* order;
  int64_t* state;
  const int64_t* state_off;
  int64_t* state_len;
  int32_t* status;
  const int32_t* list;   // heaps this launch replays (one algorithm), or null
  const uint32_t* count; // number of heaps in `list` (device), or null
  uint32_t* queue;       // heap counter (persistent mode)
  Ent* spill_free;       // per wave slot: cold free entries past LDS
  uint32_t* spill_stamp; // per wave slot: their stamps
  Ent* spill_live;       // per wave slot: cold live entries past LDS
  uint32_t* migrated;    // count of the heaps that left the lean core, or null
  int64_t n_heaps;       // heaps handled by this launch
  int64_t first;         // index into `order` of the first heap
  uint32_t cap_free, cap_live;   // total table capacities per heap
  uint32_t kf, kl;               // cold entries kept in LDS per wave
  uint32_t sf, sl;               // cold entries kept in device memory per wave
  uint32_t waves_per_group;
  uint32_t lds_wave_bytes;
  int use_queue;         // 1: pull heaps from the queue; 0: wave w takes heap w
  int64_t list_lo;       // queue mode: this launch takes list positions
  int64_t list_hi;       //   [list_lo, min(list_hi, *count))
  // ordered core from the first request (ord_any_heap): per-wave LDS pool
  // bytes, the part of it meant for chunk slots, and the device slot
  uint32_t ord_pool_bytes;
  uint32_t ord_slot_bytes;
  uint8_t* ord_dev;
  uint64_t ord_dev_stride;
  // lean core: each wave's device slot for heaps that outgrow the pool
  // (ord_spill_bytes), or null
  uint8_t* ord_spill;
  uint64_t ord_spill_stride;
  int lean_early;          // when it goes there (early_limit)
};
// ReplayParams::lean_early: only once the pool is outgrown; also once scans
// cost more; the same in the launch of the heaps taken first from the order.
enum : int { kEarlyNever = 0, kEarlyMain = 1, kEarlyHeavy = 2 };

// Validate heap parameters; on success fill the uniform heap registers.
__device__ __forceinline__ bool heap_params(const ReplayParams& p, int64_t heap, HeapRegs& h) {
  const int64_t A = p.arena[heap], g = p.align[heap];
  const int algo = p.algo[heap];
  if (algo < 0 || algo > kBitmap || g <= 0 || (g & (g - 1)) || A <= 0 || (A % g) ||
      (A / g) >= (int64_t(1) << 32))
    return false;
  h.algo = algo;
  h.arena = A;
  h.shift = (uint32_t)__builtin_ctzll((uint64_t)g);
  h.ag = (uint32_t)(A >> h.shift);
  h.status = 0;
  h.F = h.L = h.rover = h.clock = h.cnt = 0;
  return true;
}

// Whether Core's blocks may run without the checks that end a core's run
// (the lean core's tiers, the ordered core's directory).
template <typename Core>
struct UncheckedBlocks {
  static constexpr bool value = false;
};
template <int A, int R>
struct UncheckedBlocks<LeanHeap<A, R>> {
  static constexpr bool value = true;
};
template <int A, int D>
struct UncheckedBlocks<OrdHeap<A, D>> {
  static constexpr bool value = true;
};

// Whether Core may hand its heap over between two blocks of requests.
template <typename Core>
struct LeavesEarly {
  static constexpr bool value = false;
};
template <int A, int R>
struct LeavesEarly<LeanHeap<A, R>> {
  static constexpr bool value = true;
};

// Whether Core loads the next request's victim while the current one runs.
template <typename Core>
struct LooksAhead {
  static constexpr bool value = false;
};
template <int A, int D>
struct LooksAhead<OrdHeap<A, D>> {
  static constexpr bool value = true;
};

// Requests j < n of one block of 64 on core w: lane j of w0 holds request
// j's draw (free) or size in granules (allocation, 0 = larger than the
// arena), lane j of w1 its byte class (segregated fit) or its cut (free,
// other fits; read only when CUT), bit j of mfree marks the frees.  Lane j of
// `out` receives the result.  Returns the number of requests run: n, or the
// index of the request that found the lean core's tiers too small.  UNCHK:
// the core's block_safe holds for the block, so no request can find the
// tiers (or the ordered core's directory) too small, and no request of the
// block is larger than the arena, so those checks are compiled out; the only
// failure is then "nothing fits", and a result is one register per lane (the
// granule, or kNone, which no block starts at).
template <int ALGO, bool CUT, bool UNCHK, typename Core>
__device__ __forceinline__ uint32_t run_block(Core& w, uint32_t n, uint32_t w0, uint32_t w1,
                                              uint64_t mfree, uint32_t shift, int64_t& out,
                                              int32_t& st) {
  uint32_t done = n, olo = 0, ohi = 0;
  uint64_t frees = mfree;  // bit 0: the current request
  if constexpr (UNCHK && LooksAhead<Core>::value) {  // (n >= 1)
    w.next_request((uint32_t)frees & 1u, rdlane(w0, 0u));
    w.look_ahead();
  }
  for (uint32_t j = 0; j < n; ++j, frees >>= 1) {
    const uint32_t v0 = rdlane(w0, j);
    // (past the end of a last, shorter block the lanes hold copies of the last
    // request: what is loaded for them is in bounds and not used)
    if constexpr (UNCHK && LooksAhead<Core>::value)
      w.next_request(keep_scalar((uint32_t)frees) & 2u, rdlane(w0, j + 1u));
    int64_t r;
    if (keep_scalar((uint32_t)frees) & 1u) {
      if constexpr (UNCHK) r = w.template free_draw<false>(v0, CUT ? rdlane(w1, j) : 0u);
      else r = w.free_draw(v0, CUT ? rdlane(w1, j) : 0u);
    } else if (!UNCHK && v0 == 0u) {
      r = kFail;
    } else {
      if constexpr (UNCHK) r = w.template alloc<false>(v0, seg_like(ALGO) ? rdlane(w1, j) : 0u);
      else r = w.alloc(v0, seg_like(ALGO) ? rdlane(w1, j) : 0u);
    }
    if (!UNCHK && r == kOverflow) { done = j; break; }
    olo = put_lane(olo, j, (uint32_t)(uint64_t)r);
    if constexpr (!UNCHK) ohi = put_lane(ohi, j, (uint32_t)((uint64_t)r >> 32));
  }
  if constexpr (UNCHK) {
    static_assert(Core::kGranules, "a granule fits one register");
    out = olo == kNone ? kFail : (int64_t)((uint64_t)olo << shift);
  } else {
    const int64_t r = (int64_t)(((uint64_t)ohi << 32) | olo);
    out = Core::kGranules && r >= 0 ? (int64_t)((uint64_t)r << shift) : r;
    // the heap's status: its first capacity error, looked for once per block
    // rather than once per request
    if (st == 0 && ballot(lane_id() < done && r == kENoMeta) != 0ull) st = (int32_t)kENoMeta;
  }
  return done;
}

// Run requests [from, to) of `heap` on core w (either core type).  Requests
// are read 64 at a time (one per lane) and decoded by all lanes at once: a
// free carries its draw and, for the sequential fits, its cut (the fraction
// of the victim kept live, partial deallocation), an allocation its size in
// granules (0 when larger than the arena) and, for segregated fit, its byte
// class.  Loads are clamped
// to the heap's last request instead of guarded by a lane-dependent branch,
// since the values feed wave-wide reads.  Returns the position of the first
// request not run: `to`, or the request that found the lean core's tiers too
// small (it changed nothing, and the results before it are stored).
template <int ALGO, typename Core>
__device__ __forceinline__ int64_t run_requests(const ReplayParams& p, Core& w, int64_t from, int64_t to,
                                uint32_t shift, int64_t arena, int32_t& st) {
  const uint32_t lane = lane_id();
  const uint64_t gm = (1ull << shift) - 1ull;
  const int64_t last = to - 1;
  int64_t nxt = to > from ? p.req[min<int64_t>(from + lane, last)] : 0;
  for (int64_t base = from; base < to; base += 64) {
    if constexpr (LeavesEarly<Core>::value)
      if (w.F > w.leave_past && w.F <= w.leave_most) return base;
    const int64_t q = nxt;
    nxt = p.req[min<int64_t>(base + 64 + lane, last)];
    const bool is_free = q < 0;
    const bool big = q > arena;
    uint32_t sg = (uint32_t)(((uint64_t)q + gm) >> shift);
    sg = sg == 0u ? 1u : sg;
    const uint32_t w0 = is_free ? (uint32_t)~(uint64_t)q : (big ? 0u : sg);
    // segregated fit: the byte class; TLSF: the request class; the other
    // fits: a free's cut
    const uint32_t w1 = ALGO == kSegFit ? ceil_log2_u32(sg) + shift
                      : ALGO == kTlsf   ? tlsf_request_class(sg, shift)
                                        : (is_free ? (uint32_t)(~(uint64_t)q >> 32) : 0u);
    const uint64_t mfree = ballot(is_free);
    const uint32_t n = (uint32_t)min<int64_t>(64, to - base);
    int64_t out = 0;
    // a block whose frees carry no cut runs a copy with the partial-free
    // logic folded away; such a block, and one with cuts, that cannot outgrow
    // the tiers (the directory) also runs without the checks (a partial free
    // adds at most one free entry and keeps its live entry, so the block test
    // holds for it too)
    const bool cut = !seg_like(ALGO) && ballot(is_free && w1 != 0u) != 0ull;
    bool safe = false;
    if constexpr (UncheckedBlocks<Core>::value)
      safe = w.block_safe(n) && ballot(!is_free && w0 == 0u) == 0ull;
    uint32_t done = 0;
    if (cut) {
      if (safe) {
        if constexpr (UncheckedBlocks<Core>::value) {
          done = run_block<ALGO, !seg_like(ALGO), true>(w, n, w0, w1, mfree, shift, out, st);
          w.set_room();
        }
      } else {
        done = run_block<ALGO, !seg_like(ALGO), false>(w, n, w0, w1, mfree, shift, out, st);
      }
    } else if (safe) {
      if constexpr (UncheckedBlocks<Core>::value) {
        done = run_block<ALGO, false, true>(w, n, w0, w1, mfree, shift, out, st);
        w.set_room();
      }
    } else {
      done = run_block<ALGO, false, false>(w, n, w0, w1, mfree, shift, out, st);
    }
    if (lane < done) p.res[base + lane] = out;
    if (done < n) return base + done;
  }
  return to;
}

// Canonical state and status of a finished heap.
template <typename Core>
__device__ __forceinline__ void finish_heap(const ReplayParams& p, Core& w, int64_t heap,
                                            int32_t st) {
  if (p.state) {
    const int64_t so = p.state_off[heap], cap = p.state_off[heap + 1] - so;
    const int64_t need = w.dump(p.state + so, cap);
    if (lane_id() == 0) p.state_len[heap] = need;
    if (need > cap && st == 0) st = (int32_t)kERange;
  }
  if (lane_id() == 0) p.status[heap] = st;
}

template <int ALGO, int RF, int RL>
__device__ __forceinline__ void replay_heap(const ReplayParams& p, const Cold& c, const HeapRegs& regs,
                            int64_t heap) {
  WaveHeap<ALGO, RF, RL> w(c, regs, p.cap_free, p.cap_live);
  w.init();
  int32_t st = 0;
  run_requests<ALGO>(p, w, p.req_off[heap], p.req_off[heap + 1], w.h.shift, w.h.arena, st);
  finish_heap(p, w, heap, st);
}

// Requests [pos, to) of a heap on the ordered core, from an OrdHeap with one
// directory register (kept while the tables fit 64 chunks) or with all of
// them.
template <int ALGO>
__device__ __forceinline__ void ord_run(const ReplayParams& p, const OrdMem& m,
                                        OrdHeap<ALGO, 1>& w, const HeapRegs& regs, int64_t pos,
                                        int64_t to, int64_t heap, int32_t st) {
  pos = run_requests<ALGO>(p, w, pos, to, regs.shift, regs.arena, st);
  if (pos == to) {
    finish_heap(p, w, heap, st);
    return;
  }
  OrdHeap<ALGO, kOrdDir> w2(m, regs, p.cap_free, p.cap_live);
  w2.take(w);
  run_requests<ALGO>(p, w2, pos, to, regs.shift, regs.arena, st);
  finish_heap(p, w2, heap, st);
}

// Heap with invalid parameters: every result and the status are E_INVAL.
__device__ __forceinline__ void reject_heap(const ReplayParams& p, int64_t heap) {
  const uint32_t lane = lane_id();
  const int64_t b0 = p.req_off[heap], b1 = p.req_off[heap + 1];
  for (int64_t base = b0; base < b1; base += 64)
    if (base + lane < b1) p.res[base + lane] = kEInval;
  if (lane == 0) {
    p.status[heap] = (int32_t)kEInval;
    if (p.state_len) p.state_len[heap] = 0;
  }
}

// Lean path (hda_lean.h).  A heap whose tables outgrow the lean pool goes on
// from the request that did not fit: on the ordered core (hda_ordered.h) in
// the same LDS and the wave's device slot `ord`, where every request costs
// the same however large the tables are; or, without such a slot or with
// more free blocks than adopt() takes, on the general core in the wave's
// spill slot, which scans the whole table for every request.  1,000 ragged
// next-fit heaps whose tables reach thousands of entries: 17.0 ms on the
// general core, 6.5 ms on the ordered core (15,000 requests each); the
// uneven batch at the default tuning: 512 against 172 ms.
//
// Where a heap stands when it leaves the lean core.
struct LeanExit {
  enum : int32_t { kDone = 0, kOrdered = 1, kGeneral = 2 };
  int32_t next, st;
  int64_t pos;               // the first request not run
  uint32_t F, L, rover, clock;
  uint32_t cnt;              // per lane (HeapRegs::cnt)
};

// Free blocks past which a heap with few waves beside it is better off on the
// ordered core, whose request costs the same at any size, than scanning them
// 64 at a time.  Where the two cross, with pools of 20 KiB or more (at most
// two waves a SIMD): 500 first-fit heaps 9.4 ms without a limit, 7.9 / 7.3 /
// 7.0 ms at 512 / 384 / 256; 1,000 next-fit heaps in 40 KiB pools 6.1 ms, 5.3 /
// 5.2 / 5.3; 200 segregated-fit heaps 20.6 ms, 16.7 / 16.8 / 17.1; one best-fit
// heap (two sorted tables on the ordered core) 12.7 ms, 13.2 / 14.3 / 15.3.
// Pools of 10 KiB end before it matters (11.04 ms either way).
__device__ __forceinline__ constexpr uint32_t lean_max_free(int algo) {
  return algo == kFirstFit ? 256u : algo == kNextFit ? 384u : algo == kBestFit ? 1024u : 512u;
}

// The most free blocks a heap may bring to the ordered core: adopt()'s share
// of the slot, and one directory register, which describes 64 chunks (adopt()
// fills 56 entries of each, so 63 full ones leave a chunk to spare).
__device__ __forceinline__ constexpr uint32_t ord_most_free(uint32_t cap_free) {
  return ord_adopt_max(cap_free) < 56u * 63u ? ord_adopt_max(cap_free) : 56u * 63u;
}

// The limit for one launch and capacity.  It is looked at once per block of 64
// requests, each of which may add a free block, so a heap has up to limit + 64
// of them by then.  Where the ordered core does not take that many (capacities
// near the limit) leaving could end on the general core, the slowest.  The
// main launch hands over only what the ordered core takes (run_requests) and
// keeps the heap in its pool otherwise.  The heavy launch, whose pools may be
// small and whose heaps were on the ordered core from the first request before
// they started on the lean one, hands over while the ordered core still takes
// the heap.  64 heaps of small blocks in 64 KiB pools, first fit at a capacity
// of 320 free blocks / next fit at 512 / segregated fit at 640: on the general
// core 17.0 / 24.1 / 25.9 ms, on the ordered core throughout 8.2 / 9.7 / 11.0,
// now 6.9 / 7.4 / 10.3.
__device__ __forceinline__ constexpr uint32_t early_limit(int algo, uint32_t cap_free, int early) {
  const uint32_t limit = lean_max_free(algo), most = ord_most_free(cap_free);
  return early != kEarlyHeavy || limit + 64u <= most ? limit : most > 64u ? most - 64u : 0u;
}

template <int ALGO>
__device__ __forceinline__ OrdMem ord_spill_mem(const ReplayParams& p, HDA_LDS uint8_t* pool,
                                                uint32_t pool_bytes, HDA_GLOBAL uint8_t* ord) {
  return ord_mem(ALGO, pool, pool_bytes, pool_bytes / 2u, ord, p.cap_live,
                 (uint32_t)ord_area_bytes(p.cap_free));
}

// A heap on the lean core from its first request: to its end, or until its
// tables lie in the ordered core's slot (OrdHeap::stage) or in tiers c.
template <int ALGO, int RF>
__device__ __forceinline__ LeanExit lean_start(const ReplayParams& p, const LeanLds& lds,
                                               const Cold& c, int64_t heap,
                                               HDA_GLOBAL uint8_t* ord) {
  LeanExit x{LeanExit::kDone, 0, 0, 0u, 0u, 0u, 0u, 0u};
  HeapRegs h;
  if (!heap_params(p, heap, h) || h.algo != ALGO) {
    reject_heap(p, heap);
    return x;
  }
  LeanHeap<ALGO, RF> w(lds, h, p.cap_free, p.cap_live);
  w.init();
  const int64_t b1 = p.req_off[heap + 1];
  if (ord != nullptr && p.lean_early != kEarlyNever) {
    w.leave_past = early_limit(ALGO, p.cap_free, p.lean_early);
    w.leave_most = ord_most_free(p.cap_free);
  }
  x.pos = run_requests<ALGO>(p, w, p.req_off[heap], b1, w.shift, w.arena, x.st);
  if (x.pos == b1) {
    finish_heap(p, w, heap, x.st);
    return x;
  }
  if (lane_id() == 0 && p.migrated) atomicAdd(p.migrated, 1u);
  if (ord != nullptr && w.F <= ord_most_free(p.cap_free)) {
    x.next = LeanExit::kOrdered;
    OrdHeap<ALGO, 1>(ord_spill_mem<ALGO>(p, lds.base, lds.bytes, ord), h, p.cap_free,
                     p.cap_live).stage(w);
  } else {
    x.next = LeanExit::kGeneral;
    w.migrate(c, h);
    x.cnt = h.cnt;
  }
  x.F = w.F; x.L = w.L; x.rover = w.rover; x.clock = w.clock;
  return x;
}

// The rest of a heap that left the lean core for the ordered core, in the
// pool its lean tables had, or for the general core.
template <int ALGO>
__device__ __forceinline__ void ord_continue(const ReplayParams& p, const LeanLds& lds,
                                             HDA_GLOBAL uint8_t* ord, int64_t heap,
                                             const LeanExit& x) {
  HeapRegs h;
  if (!heap_params(p, heap, h)) return;  // (they were valid when the heap started)
  const OrdMem m = ord_spill_mem<ALGO>(p, lds.base, lds.bytes, ord);
  OrdHeap<ALGO, 1> o(m, h, p.cap_free, p.cap_live);
  o.adopt(x.F, x.L, x.rover, SegKey<ALGO>::kShift);
  ord_run<ALGO>(p, m, o, h, x.pos, p.req_off[heap + 1], heap, x.st);
}
template <int ALGO>
__device__ __forceinline__ void general_continue(const ReplayParams& p, const Cold& c,
                                                 int64_t heap, const LeanExit& x) {
  HeapRegs h;
  if (!heap_params(p, heap, h)) return;
  h.F = x.F; h.L = x.L; h.rover = x.rover; h.clock = x.clock; h.cnt = x.cnt;
  WaveHeap<ALGO, 0, 0> g(c, h, p.cap_free, p.cap_live);
  int32_t st = x.st;
  run_requests<ALGO>(p, g, x.pos, p.req_off[heap + 1], h.shift, h.arena, st);
  finish_heap(p, g, heap, st);
}

// Lean replay of one heap known to use algorithm ALGO, all of it in place
// (the GPU kernels call the three parts out of line, hda_replay.hip).
template <int ALGO, int RF>
__device__ __forceinline__ void lean_one_heap(const ReplayParams& p, const LeanLds& lds,
                                              const Cold& c, int64_t heap,
                                              HDA_GLOBAL uint8_t* ord = nullptr) {
  const LeanExit x = lean_start<ALGO, RF>(p, lds, c, heap, ord);
  if (x.next == LeanExit::kOrdered) ord_continue<ALGO>(p, lds, ord, heap, x);
  if (x.next == LeanExit::kGeneral) general_continue<ALGO>(p, c, heap, x);
}

// Any algorithm (used where one program must serve every heap).
template <int RF, int RL>
__device__ void replay_any_heap(const ReplayParams& p, const Cold& c, int64_t heap) {
  HeapRegs h;
  if (!heap_params(p, heap, h)) {
    reject_heap(p, heap);
    return;
  }
  switch (h.algo) {
    case kFirstFit: replay_heap<kFirstFit, RF, RL>(p, c, h, heap); break;
    case kNextFit: replay_heap<kNextFit, RF, RL>(p, c, h, heap); break;
    case kBestFit: replay_heap<kBestFit, RF, RL>(p, c, h, heap); break;
    case kSegFit: replay_heap<kSegFit, RF, RL>(p, c, h, heap); break;
    case kTlsf: replay_heap<kTlsf, RF, RL>(p, c, h, heap); break;
    default: reject_heap(p, heap); break;  // the bitmask allocator has its own kernel
  }
}

// Ordered core (hda_ordered.h) for one heap from its first request (the CPU
// emulation's way in; the kernels reach the core through ord_continue):
// tables in the wave's LDS pool and, past it, in its device slot.
template <int ALGO>
__device__ __forceinline__ void ord_replay_heap(const ReplayParams& p, HDA_LDS uint8_t* pool,
                                HDA_GLOBAL uint8_t* dev, const HeapRegs& regs, int64_t heap) {
  const OrdMem m = ord_mem(ALGO, pool, p.ord_pool_bytes, p.ord_slot_bytes, dev, p.cap_live);
  OrdHeap<ALGO, 1> w(m, regs, p.cap_free, p.cap_live);
  w.init();
  ord_run<ALGO>(p, m, w, regs, p.req_off[heap], p.req_off[heap + 1], heap, 0);
}

__device__ __forceinline__ void ord_any_heap(const ReplayParams& p, HDA_LDS uint8_t* pool,
                                             HDA_GLOBAL uint8_t* dev, int64_t heap) {
  HeapRegs h;
  if (!heap_params(p, heap, h)) {
    reject_heap(p, heap);
    return;
  }
  switch (h.algo) {
    case kFirstFit: ord_replay_heap<kFirstFit>(p, pool, dev, h, heap); break;
    case kNextFit: ord_replay_heap<kNextFit>(p, pool, dev, h, heap); break;
    case kBestFit: ord_replay_heap<kBestFit>(p, pool, dev, h, heap); break;
    case kSegFit: ord_replay_heap<kSegFit>(p, pool, dev, h, heap); break;
    case kTlsf: ord_replay_heap<kTlsf>(p, pool, dev, h, heap); break;
    default: reject_heap(p, heap); break;  // the bitmask allocator has its own kernel
  }
}

// Bitmask-allocator replay of one heap from its table of free blocks in the
// wave's LDS pool; a heap whose tables outgrow the pool continues on the
// flags (hda_bitmap.h) in the wave's workspace slot, the first kn summaries
// and kl live entries in the same LDS.
//
// Where a heap stands when it leaves the table: the first request not run,
// and the table, whose first chunks (fa, fe: per lane) are in registers and
// whose rest and live entries are still in the pool.
struct BitmapExit {
  int32_t next, st;      // next: 0 the heap is finished, 1 it goes on on the flags
  int64_t pos;
  uint32_t F, L, rover;
  uint32_t fa[kBitmapRF], fe[kBitmapRF];
};

__device__ __forceinline__ BitmapExit bitmap_start(const ReplayParams& p, const LeanLds& lds,
                                                   uint64_t max_granules, int64_t heap) {
  BitmapExit x{};
  HeapRegs h;
  if (!heap_params(p, heap, h) || h.algo != kBitmap || (uint64_t)h.ag > max_granules) {
    reject_heap(p, heap);
    return x;
  }
  LeanHeap<kBitmap, kBitmapRF> w(lds, h, kNone, p.cap_live);
  w.init();
  const int64_t b1 = p.req_off[heap + 1];
  x.pos = run_requests<kBitmap>(p, w, p.req_off[heap], b1, h.shift, h.arena, x.st);
  if (x.pos == b1) {
    finish_heap(p, w, heap, x.st);
    return x;
  }
  if (lane_id() == 0 && p.migrated) atomicAdd(p.migrated, 1u);
  x.next = 1;
  x.F = w.F; x.L = w.L; x.rover = w.rover;
#pragma unroll
  for (int k = 0; k < kBitmapRF; ++k) { x.fa[k] = w.fa[k]; x.fe[k] = w.fe[k]; }
  return x;
}

__device__ __forceinline__ void bitmap_continue(const ReplayParams& p, const LeanLds& lds,
                                                uint64_t* bits, uint64_t* nodes, Ent* live,
                                                uint32_t kn, int64_t heap, const BitmapExit& x) {
  HeapRegs h;
  if (!heap_params(p, heap, h)) return;  // (they were valid when the heap started)
  LeanHeap<kBitmap, kBitmapRF> w(lds, h, kNone, p.cap_live);
  w.F = x.F; w.L = x.L; w.rover = x.rover;
#pragma unroll
  for (int k = 0; k < kBitmapRF; ++k) { w.fa[k] = x.fa[k]; w.fe[k] = x.fe[k]; }
  BitHeap b(bits, nodes, live, (HDA_LDS uint64_t*)lds.base, kn,
            (HDA_LDS Ent*)(lds.base + 8u * kn), (lds.bytes - 8u * kn) / 8u, h, p.cap_live);
  b.take(w);
  int32_t st = x.st;
  run_requests<kBitmap>(p, b, x.pos, p.req_off[heap + 1], h.shift, h.arena, st);
  finish_heap(p, b, heap, st);
}

// Both parts in place (the GPU kernel calls them out of line, hda_bitmap.hip).
__device__ __forceinline__ void bitmap_lean_heap(const ReplayParams& p, const LeanLds& lds,
                                                 uint64_t* bits, uint64_t* nodes, Ent* live,
                                                 uint32_t kn, uint64_t max_granules,
                                                 int64_t heap) {
  const BitmapExit x = bitmap_start(p, lds, max_granules, heap);
  if (x.next) bitmap_continue(p, lds, bits, nodes, live, kn, heap, x);
}

// Bitmask-allocator replay of one heap (hda_bitmap.h) in a workspace slot
// of max_granules flags, their node summaries and p.cap_live live entries
// (the first kn summaries and kl live entries in the wave's LDS instead); a
// heap of another algorithm or a larger arena is rejected.
__device__ __forceinline__ void bitmap_one_heap(const ReplayParams& p, uint64_t* bits,
                                                uint64_t* nodes, Ent* live,
                                                HDA_LDS uint64_t* lnodes, uint32_t kn,
                                                HDA_LDS Ent* llive, uint32_t kl,
                                                uint64_t max_granules, int64_t heap) {
  HeapRegs h;
  if (!heap_params(p, heap, h) || h.algo != kBitmap || (uint64_t)h.ag > max_granules) {
    reject_heap(p, heap);
    return;
  }
  BitHeap w(bits, nodes, live, lnodes, kn, llive, kl, h, p.cap_live);
  w.init();
  int32_t st = 0;
  run_requests<kBitmap>(p, w, p.req_off[heap], p.req_off[heap + 1], h.shift, h.arena, st);
  finish_heap(p, w, heap, st);
}

}  // namespace hda
