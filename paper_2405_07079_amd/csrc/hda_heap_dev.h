// A heap whose state persists between launches.  Its device-memory layout: a
// header holding the wave-uniform registers and the per-class counts,
// followed by the free table, its push stamps and the live table.  And one
// call on such a heap by one wave (the kernel of hda_heap.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hda_core.h"

namespace hda {

struct HeapHdr {
  uint32_t F, L, ag, shift, rover, clock;
  int32_t algo, status;
  int64_t arena;
  uint32_t cf, cl;          // table capacities (multiples of 64)
  uint32_t pad[4];
  uint32_t cnt[64];         // free blocks per byte class
};
static_assert(sizeof(HeapHdr) % 16 == 0, "header keeps the tables 16 B aligned");

__host__ __device__ inline size_t heap_bytes(uint32_t cf, uint32_t cl) {
  return sizeof(HeapHdr) + (size_t)cf * 8 + (size_t)cf * 4 + (size_t)cl * 8;
}

__device__ inline Cold heap_cold(HeapHdr* hd) {
  uint8_t* base = reinterpret_cast<uint8_t*>(hd) + sizeof(HeapHdr);
  Cold c;
  c.lf = nullptr; c.lst = nullptr; c.ll = nullptr;  // no LDS part
  c.kf = 0; c.kl = 0;
  c.cf = hd->cf; c.cl = hd->cl;
  c.gf = (HDA_GLOBAL Ent*)(base);
  c.gst = (HDA_GLOBAL uint32_t*)(base + (size_t)c.cf * 8);
  c.gl = (HDA_GLOBAL Ent*)(base + (size_t)c.cf * 12);
  return c;
}

__device__ inline HeapRegs load_regs(const HeapHdr* hd) {
  HeapRegs h;
  h.F = hd->F; h.L = hd->L; h.ag = hd->ag; h.shift = hd->shift;
  h.rover = hd->rover; h.clock = hd->clock; h.algo = hd->algo; h.status = hd->status;
  h.arena = hd->arena;
  h.cnt = hd->cnt[lane_id()];
  return h;
}

__device__ inline void store_regs(HeapHdr* hd, const HeapRegs& h) {
  hd->cnt[lane_id()] = h.cnt;
  if (lane_id() == 0) {
    hd->F = h.F; hd->L = h.L; hd->rover = h.rover; hd->clock = h.clock;
    hd->status = h.status;
  }
}

enum : int { kOpInit = 0, kOpAlloc = 1, kOpFree = 2, kOpDump = 3, kOpFreePartial = 4 };

// The caller's host thread returns as soon as it sees `r` in *word, so the
// heap's tables and registers are stored first and the word is released at
// system scope after them: a call that has returned has nothing left to do on
// the device but end its kernel, not even to write the heap's lines back, and
// its memory may be given to others without a wait for the stream.
__device__ inline void publish(int64_t* word, int64_t r) {
  wave_sync();  // (every lane has stored its part)
  if (lane_id() == 0) __hip_atomic_store(word, r, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int ALGO>
__device__ void heap_call_t(HeapHdr* hd, int op, int64_t arg, int64_t* dump, int64_t cap,
                            int64_t* word) {
  const Cold c = heap_cold(hd);
  WaveHeap<ALGO, 0, 0> w(c, load_regs(hd), hd->cf, hd->cl);
  int64_t r = 0;
  if (op == kOpInit) {
    w.init();
  } else if (op == kOpAlloc) {
    r = arg < 0 ? kEInval : w.alloc_bytes(arg);
  } else if (op == kOpFree) {
    r = w.free_offset(arg);
  } else if (op == kOpFreePartial) {
    r = w.free_partial(arg);
  } else {
    r = w.dump(dump, cap);
  }
  store_regs(hd, w.h);
  publish(word, r);
}

}  // namespace hda
