// Lean replay core: one wavefront replays one heap with exactly two storage
// tiers.  Free-table entry i lives in lane i % 64 of 64-entry chunk i / 64;
// the first RF chunks are VGPRs and the rest LDS.  The wave's LDS region is
// one pool shared by both tables: free chunks from its start, live entries
// from its end, so a heap with many free blocks and one with many live
// blocks both fit.  Selection (Sec. II, Sec. IV, Sec. V-A) and the
// neighbour search of coalescing (Alg. 2, Alg. 5) are wave-wide scans over the
// chunks followed by one DPP reduction.
//
// Unused free slots hold address ~0 and end ~0.  Such a slot never fits a
// request (every request is at least one granule) and never borders a block
// (no block starts at granule ~0; the one block that can end there, in an
// arena of 2^32 - 1 granules, is matched by its start instead), so every
// scan covers whole chunks with no bounds mask.
//
// What bounds it: a heap is a chain of dependent requests, and four waves per
// SIMD keep the vector and scalar units busy with table arithmetic (HBM, 16 B
// per request, is idle by comparison), so the instructions per request set
// the rate.  Keeping ends instead of sizes, one branch and one access per
// field instead of selects over every register chunk, two LDS chunks scanned
// without a loop, results kept as 32-bit granules until the block is stored,
// and the entry that fills a live hole never made uniform took 4,096 heaps x
// 100,000 requests (16 MiB, 64 B) from 53.7 to 38.7 ms on best fit and from
// 64.3 to 48.7 ms on segregated fit, and a lone first-fit heap of 64 KiB from
// 271 to 207 ns a request.  (Tried and not kept: keys of a chunk together
// after its blocks; one or four register chunks; the next free's victim
// loaded ahead, 5-8 % slower even for a lone heap; entries found by a scan
// kept as chunk and lane.)
//
// When the tables would outgrow the pool before reaching the capacities the
// caller asked for, the request stops with kOverflow (changing nothing) and
// the heap goes on with its tables in the ordered core (hda_ordered.h) or in
// the general core (hda_core.h), both of which continue into device memory.
// Results are the same on every path.
//
// Same rules as the general core: values that feed a cross-lane operation are
// never produced under a lane-dependent branch, and every LDS access is
// preceded by wave_sync().
#pragma once
#include <stdint.h>

#include "hda_core.h"

namespace hda {

constexpr int64_t kOverflow = -100;      // internal: the fast tiers are too small
// Segregated-fit key of a free block: the block's class in the top bits
// (6 for the 64 byte classes of segregated fit, 11 for the 2,048 classes of
// TLSF) and, below, the push stamp taken from the all-ones value (limit - 1 -
// stamp).  The smallest key at or above c << shift is then the head (the
// block pushed last) of the first non-empty class at or above c, so one
// wave-wide minimum does Alg. 4's class search (TLSF: the two-level bitmap
// lookup of Sec. V-B) and the list-head lookup together, and no per-class
// counts are kept on the request path.  Stamps start at 1, so a key never
// equals kNone, the key of an empty slot.
template <int ALGO>
struct SegKey {
  static constexpr uint32_t kShift = ALGO == kTlsf ? 21u : 26u;
  static constexpr uint32_t kLimit = 1u << kShift;   // stamps below this
  static constexpr uint32_t kMask = kLimit - 1u;
  static constexpr uint32_t kClasses = ALGO == kTlsf ? kTlsfClasses : 64u;
};

// A wave-uniform value kept on the scalar unit: the compiler may not fold it
// into a carry or population-count idiom that it evaluates per lane.
__device__ __forceinline__ uint32_t keep_scalar(uint32_t v) {
#ifdef __HIP_DEVICE_COMPILE__
  asm("" : "+s"(v));
#endif
  return v;
}

// The wave's LDS pool: `bytes` (a multiple of 16) from `base`.
struct LeanLds {
  HDA_LDS uint8_t* base;
  uint32_t bytes;
};

// Free entries hold a block's address and its end (the granule past it): an
// allocation is cut from the low end, so it rewrites only the address, a
// merge to the left only the end, a merge to the right only the address, and
// the neighbour search compares both as they are.
// In LDS an entry is 8 bytes (address in the low word, end in the high
// word), with segregated fit's key and a pad word after it: 16 bytes, so that
// one shift finds any of them.  (The keys of a chunk kept together after its
// blocks met no bank conflicts but cost more address arithmetic: 10.70 ms
// against 10.45 ms for 4,096 heaps x 20,000 requests.)
// Fields of a free entry a write touches (the key goes with either).
enum : int { kAddr = 1, kEnd = 2, kBoth = 3 };

// One word of an 8-byte entry (may alias it).
typedef uint32_t __attribute__((may_alias)) half_t;

template <int ALGO, int RF>
struct LeanHeap {
  static constexpr bool kSeg = ALGO == kSegFit || ALGO == kTlsf;
  static constexpr bool kRover = ALGO == kNextFit || ALGO == kBitmap;
  static constexpr uint32_t kKeyShift = SegKey<ALGO>::kShift;
  static constexpr uint32_t kStampLimit = SegKey<ALGO>::kLimit;
  static constexpr uint32_t kStampMask = SegKey<ALGO>::kMask;
  static constexpr uint32_t kClasses = SegKey<ALGO>::kClasses;
  static constexpr uint32_t HF = 64u * RF;
  static_assert(RF >= 1, "at least one register chunk");

  LeanLds m;
  uint32_t fa[RF], fe[RF], fk[RF];  // address, end, segregated-fit key
  int64_t arena;
  uint32_t shift, ag;
  static constexpr bool kGranules = true;  // alloc / free_draw return granules
  uint32_t F, L, rover, clock;
  uint32_t hint;                  // next fit, bitmask: the entry last cut (it may have moved)
  // The numbers of the first two LDS chunks in registers of their own: as
  // constants the compiler puts them where a select needs the opposite
  // comparison, and compares twice (best fit 1.8 %, segregated fit 0.7 %
  // faster; first fit 0.5 % slower, which takes constants).
  static constexpr bool kColdId = ALGO == kBestFit || kSeg;
  uint32_t cold_id[2];
  uint32_t leave_past = kNone, leave_most = 0u;  // hand the heap over with more free blocks
                                                 // than the first, but not the second
  uint32_t capF, capL;            // the caller's capacities (E_NOMETA past them)
  uint32_t live_room;             // live entries the pool holds beside the current free chunks

  __device__ __forceinline__ LeanHeap(const LeanLds& lds, const HeapRegs& h, uint32_t cap_free,
                                      uint32_t cap_live)
      : m(lds), arena(h.arena), shift(h.shift), ag(h.ag),
        cold_id{opaque((uint32_t)RF), opaque((uint32_t)RF + 1u)}, capF(cap_free),
        capL(cap_live) {}

  // ---- the LDS pool ----
  static constexpr uint32_t kRec = kSeg ? 16u : 8u;  // bytes per free entry in LDS
  // Pool bytes the tables take with f free and l live entries: the free
  // entries past the register chunks in whole 64-entry chunks (scans read
  // whole chunks), then the live entries.
  __device__ __forceinline__ uint32_t need_bytes(uint32_t f, uint32_t l) const {
    const uint32_t cold = f > HF ? f - HF : 0u;
    return ((cold + 63u) & ~63u) * kRec + l * 8u;
  }
  // Recompute live_room after F changed.
  __device__ __forceinline__ void set_room() {
    const uint32_t cold = F > HF ? F - HF : 0u;
    const uint32_t used = ((cold + 63u) & ~63u) * kRec;
    live_room = used <= m.bytes ? (m.bytes - used) >> 3 : 0u;
  }
  // LDS free entry j (free-table index, j >= HF; per lane or wave-uniform).
  __device__ __forceinline__ HDA_LDS Ent* cold_at(uint32_t j) const {
    return (HDA_LDS Ent*)(m.base + (j * kRec - HF * kRec));
  }
  __device__ __forceinline__ static void cold_load(const HDA_LDS Ent* at, uint32_t& a,
                                                   uint32_t& e, uint32_t& k) {
    const Ent v = at[0];
    a = (uint32_t)v; e = (uint32_t)(v >> 32);
    k = kSeg ? ((const HDA_LDS half_t*)at)[2] : 0u;
  }
  __device__ __forceinline__ void cold_get(uint32_t j, uint32_t& a, uint32_t& e,
                                           uint32_t& k) const {
    cold_load(cold_at(j), a, e, k);
  }
  template <int FIELDS>
  __device__ __forceinline__ void cold_put(uint32_t j, uint32_t a, uint32_t e,
                                           uint32_t k) const {
    HDA_LDS Ent* at = cold_at(j);
    if constexpr (FIELDS == kBoth) at[0] = ((uint64_t)e << 32) | a;
    else ((HDA_LDS half_t*)at)[FIELDS == kEnd ? 1 : 0] = FIELDS == kEnd ? e : a;
    if constexpr (kSeg) ((HDA_LDS half_t*)at)[2] = k;
  }
  // This lane's entry of LDS chunk c (c >= RF).
  __device__ __forceinline__ void chunk_get(uint32_t c, uint32_t& a, uint32_t& e,
                                            uint32_t& k) const {
    cold_load((const HDA_LDS Ent*)(m.base + ((c - RF) * 64u + lane_id()) * kRec), a, e, k);
  }
  // Live entry i, counted from the end of the pool.
  __device__ __forceinline__ HDA_LDS Ent* live_ptr(uint32_t i) const {
    return (HDA_LDS Ent*)(m.base + (m.bytes - 8u)) - i;
  }

  // the list a free block of sg granules belongs to
  __device__ __forceinline__ uint32_t list_class(uint32_t sg) const {
    return ALGO == kTlsf ? tlsf_class(sg, shift) : floor_log2_u32(sg) + shift;
  }
  __device__ __forceinline__ uint32_t seg_key(uint32_t sg) {
    return (list_class(sg) << kKeyShift) | (clock++ ^ kStampMask);
  }
  // Segregated fit, lane k: the number of free blocks of byte class k (for
  // the canonical state and the hand-over to the general core; not kept per
  // request).
  __device__ uint32_t class_counts() {
    uint32_t n = 0;
    for (uint32_t j = 0; j < F; ++j) {
      uint32_t a, e, k;
      read(j, a, e, k);
      n += lane_id() == (k >> kKeyShift) ? 1u : 0u;
    }
    return n;
  }

  // ---- free-table entries by wave-uniform index ----
  // A register chunk is chosen by a branch, like write()'s: one read per
  // field instead of one per chunk and a select.
  template <int K = 0>
  __device__ __forceinline__ void read(uint32_t j, uint32_t& a, uint32_t& e, uint32_t& k) {
    if constexpr (K < RF) {
      if (j < 64u * (K + 1)) {
        a = rdlane(fa[K], j & 63u);
        e = rdlane(fe[K], j & 63u);
        k = kSeg ? rdlane(fk[K], j & 63u) : 0u;
      } else {
        read<K + 1>(j, a, e, k);
      }
    } else {
      wave_sync();
      uint32_t ea, ee, ek;
      cold_get(j, ea, ee, ek);
      a = uniform(ea);
      e = uniform(ee);
      k = kSeg ? uniform(ek) : 0u;
    }
  }
  // The block (address, end) of free entry j.
  __device__ __forceinline__ void read_block(uint32_t j, uint32_t& a, uint32_t& e) {
    uint32_t k;
    read(j, a, e, k);
  }
  __device__ __forceinline__ uint32_t addr_at(uint32_t j) {
    uint32_t a, e;
    read_block(j, a, e);
    return a;
  }
  __device__ __forceinline__ uint32_t end_at(uint32_t j) {
    uint32_t a, e;
    read_block(j, a, e);
    return e;
  }
  // Write fields of entry j (segregated fit: and its key).  A register chunk
  // is chosen by a branch and takes one write per field.  An LDS entry is
  // stored by every lane with the same value: a store guarded by a lane test
  // would be merged by the optimiser with the uniform test around it into
  // one divergent branch, which turns the heap's counters into per-lane
  // values.
  template <int FIELDS, int K = 0>
  __device__ __forceinline__ void write(uint32_t j, uint32_t a, uint32_t e, uint32_t k) {
    if constexpr (K < RF) {
      if (j < 64u * (K + 1)) {
        if constexpr (FIELDS & kAddr) fa[K] = put_lane(fa[K], j, a);
        if constexpr (FIELDS & kEnd) fe[K] = put_lane(fe[K], j, e);
        if constexpr (kSeg) fk[K] = put_lane(fk[K], j, k);
      } else {
        write<FIELDS, K + 1>(j, a, e, k);
      }
    } else {
      wave_sync();
      cold_put<FIELDS>(j, a, e, k);
    }
  }
  // ---- live table ----
  __device__ __forceinline__ void live_write(uint32_t i, uint32_t a, uint32_t s) {
    wave_sync();
    *live_ptr(i) = mk_ent(a, s);  // every lane, same value (see write())
  }

  // Visit every chunk holding entries: f(chunk, a, e, key).  The first two
  // LDS chunks, where most scans end, are at fixed places; later ones are
  // loaded four at a time before any is used, so their latencies overlap.
  template <int N, typename Fn>
  __device__ __forceinline__ void scan_cold(uint32_t c, Fn&& f) const {
    wave_sync();
    uint32_t ea[N], ee[N], ek[N];
#pragma unroll
    for (int u = 0; u < N; ++u) chunk_get(c + u, ea[u], ee[u], ek[u]);
#pragma unroll
    for (int u = 0; u < N; ++u)
      f(kColdId && N <= 2 && c == (uint32_t)RF ? cold_id[u & 1] : c + u, ea[u], ee[u], ek[u]);
  }
  template <typename Fn>
  __device__ __forceinline__ void scan(Fn&& f) {
#pragma unroll
    for (int k = 0; k < RF; ++k) f((uint32_t)k, fa[k], fe[k], kSeg ? fk[k] : 0u);
    if (F <= HF) return;
    if (F <= HF + 64u) {
      scan_cold<1>(RF, f);
      return;
    }
    scan_cold<2>(RF, f);
    uint32_t c = RF + 2;
    for (; 64u * (c + 3u) < F; c += 4u) scan_cold<4>(c, f);
    for (; 64u * c < F; ++c) scan_cold<1>(c, f);
  }

  // The same one chunk at a time, for work done once per heap (one copy of f
  // for the LDS chunks).
  template <typename Fn>
  __device__ __forceinline__ void each_chunk(Fn&& f) const {
#pragma unroll
    for (int k = 0; k < RF; ++k) f((uint32_t)k, fa[k], fe[k], kSeg ? fk[k] : 0u);
    for (uint32_t c = RF; 64u * c < F; ++c) scan_cold<1>(c, f);
  }

  // Alg. 6: one free block [0, A).
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int k = 0; k < RF; ++k) { fa[k] = kNone; fe[k] = kNone; fk[k] = kNone; }
    F = 1; L = 0; rover = 0; clock = 1; hint = 0;
    set_room();
    write<kBoth>(0, 0u, ag, kSeg ? seg_key(ag) : 0u);
  }

  // Read entry j and clear its slot.
  template <int K = 0>
  __device__ __forceinline__ void take_out(uint32_t j, uint32_t& a, uint32_t& e, uint32_t& k) {
    if constexpr (K < RF) {
      if (j < 64u * (K + 1)) {
        a = rdlane(fa[K], j & 63u);
        e = rdlane(fe[K], j & 63u);
        fa[K] = put_lane(fa[K], j, kNone);
        fe[K] = put_lane(fe[K], j, kNone);
        if constexpr (kSeg) {
          k = rdlane(fk[K], j & 63u);
          fk[K] = put_lane(fk[K], j, kNone);
        }
      } else {
        take_out<K + 1>(j, a, e, k);
      }
    } else {
      read<RF>(j, a, e, k);
      wave_sync();
      cold_put<kBoth>(j, kNone, kNone, kNone);
    }
  }
  // Remove free entry j: the last entry is taken out of its slot and moves
  // into j's place.
  template <bool CHK = true>
  __device__ __forceinline__ void remove(uint32_t j) {
    const uint32_t last = F - 1u;
    uint32_t a, e, k = 0;
    take_out(last, a, e, k);
    if (j != last) write<kBoth>(j, a, e, k);
    F = last;
    if (CHK) set_room();
  }

  // Append a free entry (the caller has checked the pool and the capacity).
  template <bool CHK = true, int K = 0>
  __device__ __forceinline__ void append(uint32_t a, uint32_t e, uint32_t k) {
    if constexpr (K < RF) {
      if (F < 64u * (K + 1)) {
        fa[K] = put_lane(fa[K], F, a);
        fe[K] = put_lane(fe[K], F, e);
        if constexpr (kSeg) fk[K] = put_lane(fk[K], F, k);
        ++F;
        if (CHK) set_room();
      } else {
        append<CHK, K + 1>(a, e, k);
      }
    } else {
      if ((F & 63u) == 0u) {  // a new LDS chunk: its slots start empty
        wave_sync();
        cold_put<kBoth>(F + lane_id(), kNone, kNone, kNone);
      }
      wave_sync();
      cold_put<kBoth>(F, a, e, k);
      ++F;
      if (CHK) set_room();
    }
  }

  // Bitmask allocator (Sec. III-B, one flag per granule, searched from the
  // rover): the free runs of the flags are exactly the free blocks, so its
  // answers follow from the table.  The run taken starts at the lowest
  // p >= rover with sg free granules in a row -- max(address, rover) of some
  // block -- else at the lowest address of a block that fits.  p is the first
  // granule taken, (a, e) the block it lies in.
  //
  // The block that holds the rover comes first in that order, and after an
  // allocation it is the remainder the last one left, so its entry is tried
  // before the scan.  An entry that moved meanwhile fails the test below
  // (free blocks do not overlap: a block holding the rover is the one that
  // does) and the scan decides.
  __device__ __forceinline__ bool select_run(uint32_t sg, uint32_t& j, uint32_t& a, uint32_t& e,
                                             uint32_t& p) {
    if (hint < F) {
      read_block(hint, a, e);
      if (rover - a < e - a && e - rover >= sg) {
        j = hint;
        p = rover;
        return true;
      }
    }
    uint32_t best = kNone, bc = 0;
    scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
      const uint32_t st = ea > rover ? ea : rover;
      const uint32_t past = ee > st ? ee - st : 0u;  // granules from the rover on
      const uint32_t t = ee - ea >= sg ? (past >= sg ? st : ea) - rover : kNone;
      const bool lt = t < best;
      best = lt ? t : best;
      bc = lt ? c : bc;
    });
    const uint32_t K = wave_min(best);
    uint64_t mk;
    if (K != kNone) {
      mk = ballot(best == K);
    } else {
      // a block starting right below the rover has key ~0 as well
      uint64_t any = 0ull;
      scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
        const bool hit = ee - ea >= sg && ea + 1u == rover;
        any |= ballot(hit);
        bc = hit ? c : bc;
      });
      if (any == 0ull) return false;
      mk = any;
    }
    const uint32_t l = ctz64(mk);
    j = 64u * rdlane(bc, l) + l;
    p = K + rover;
    read_block(j, a, e);
    return true;
  }

  // Selection.  On success j is the chosen entry, a its block's address and
  // s its size.
  __device__ __forceinline__ bool select(uint32_t sg, uint32_t kreq, uint32_t& j, uint32_t& a,
                                         uint32_t& s) {
    if constexpr (ALGO == kFirstFit || ALGO == kNextFit) {
      if constexpr (ALGO == kNextFit) {
        // The block that holds the rover is the first one ending past it;
        // after an allocation it is the remainder the last one left, so its
        // entry is tried before the scan (an entry that moved meanwhile
        // fails the test: free blocks do not overlap).
        if (hint < F) {
          uint32_t e;
          read_block(hint, a, e);
          s = e - a;
          if (rover - a < s && s >= sg) {
            j = hint;
            return true;
          }
        }
      }
      // first fit: lowest address among blocks that fit.  Next fit: blocks
      // are taken in cyclic order starting at the first whose end is past the
      // rover; since free blocks do not overlap, that order is the order of
      // end - rover - 1 taken mod 2^32.  The block ending exactly at the rover
      // (last in that order) has key ~0, which the scan cannot tell from
      // "none", so it is looked for separately when nothing else fits.
      const uint32_t nr = ~rover;
      uint32_t best = kNone, bc = 0, bsz = 0;  // bsz: the candidate's size
      scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
        const uint32_t es = ee - ea;
        const uint32_t t = es >= sg ? (ALGO == kFirstFit ? ea : ee + nr) : kNone;
        const bool lt = t < best;
        best = lt ? t : best;
        bc = lt ? c : bc;
        bsz = lt ? es : bsz;
      });
      const uint32_t K = wave_min(best);
      uint64_t mk;
      uint32_t end;  // next fit: end of the chosen block
      if (K != kNone) {
        mk = ballot(best == K);
        end = K - nr;
      } else {
        if (ALGO == kFirstFit) return false;
        uint64_t any = 0ull;
        scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
          const bool hit = ee - ea >= sg && ee == rover;
          any |= ballot(hit);
          bc = hit ? c : bc;
          bsz = hit ? ee - ea : bsz;
        });
        if (any == 0ull) return false;
        mk = any;
        end = rover;
      }
      const uint32_t l = ctz64(mk);
      j = 64u * rdlane(bc, l) + l;
      s = rdlane(bsz, l);
      a = ALGO == kFirstFit ? K : end - s;
      return true;
    } else if constexpr (ALGO == kBestFit) {
      // smallest size, then lowest address: (leftover, address) compared as
      // one 64-bit value, one vector compare per chunk.  The leftover is
      // size - sg mod 2^32: a block that fits leaves at most ~sg, one that
      // does not (empty slots included, size 0) wraps to more, so no test
      // of the size is needed per entry.
      uint64_t best = ~0ull;
      uint32_t bc = 0;
      scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
        const uint64_t key = ((uint64_t)(ee - ea - sg) << 32) | ea;
        const bool take = key < best;
        best = take ? key : best;
        bc = take ? c : bc;
      });
      const uint32_t bs = (uint32_t)(best >> 32), ba = (uint32_t)best;
      const uint32_t K = wave_min(bs);
      if (K > keep_scalar(~sg)) return false;
      uint64_t mk = ballot(bs == K);
      if (keep_scalar((uint32_t)__builtin_popcountll(mk)) > 1u) {
        const uint32_t A2 = wave_min(bs == K ? ba : kNone);
        mk = ballot(bs == K && ba == A2);
      }
      const uint32_t l = ctz64(mk);
      j = 64u * rdlane(bc, l) + l;
      a = rdlane(ba, l);
      s = K + sg;
      return true;
    } else {
      // segregated fit: the first non-empty class at or above the request's,
      // and in it the block pushed last (Alg. 4): the smallest key at or
      // above the request's class
      // (a request no larger than the arena has a class below kClasses:
      // arenas are below 2^63 bytes, and TLSF's rounding stays at 2^63)
      const uint32_t lo = kreq << kKeyShift;
      // Keys are compared as (key - lo) mod 2^32: keys below lo wrap past
      // every key at or above it and past the empty slots' key ~0 (which
      // maps to ~lo), so the smallest such value is the smallest key at or
      // above lo whenever it is below ~lo.  Only the chunk is carried; the
      // block is read from the chosen slot afterwards.
      uint32_t best = kNone, bc = 0;
      scan([&](uint32_t ch, uint32_t, uint32_t, uint32_t ek) {
        const uint32_t t = ek - lo;
        const bool lt = t < best;
        best = lt ? t : best;
        bc = lt ? ch : bc;
      });
      const uint32_t K = wave_min(best);
      if (K >= keep_scalar(~lo)) return false;
      const uint32_t l = ctz64(ballot(best == K));
      j = 64u * rdlane(bc, l) + l;
      uint32_t e;
      read_block(j, a, e);
      s = e - a;
      return true;
    }
  }

  // Allocate sg granules; kreq is the request's byte class (segregated fit).
  // Returns the first granule, -1, kENoMeta or kOverflow.
  // CHK = false: the caller has established that no request of the current
  // block can outgrow the tiers or reach the capacities (block_safe), so
  // those checks and the upkeep of live_room are left out; live_room is
  // refreshed after the block.
  template <bool CHK = true>
  __device__ __forceinline__ int64_t alloc(uint32_t sg, uint32_t kreq) {
    uint32_t j = 0, a = 0, s = 0;
    if constexpr (ALGO == kBitmap) {
      uint32_t p = 0, e = 0;
      if (!select_run(sg, j, a, e, p)) return kFail;
      if (CHK && L >= capL) return kENoMeta;
      if (CHK && L >= live_room) return kOverflow;
      // the part below p stays, the part above the run is the new remainder
      const uint32_t pe = p + sg;
      if (p == a) {
        hint = j;
        if (pe != e) write<kAddr>(j, pe, 0u, 0u);
        else remove<CHK>(j);
      } else {
        if (pe != e) {
          if (CHK && need_bytes(F + 1u, L + 1u) > m.bytes) return kOverflow;
          hint = F;
          append<CHK>(pe, e, 0u);
        }
        write<kEnd>(j, 0u, p, 0u);
      }
      live_write(L, p, sg);
      ++L;
      rover = pe;
      return (int64_t)(uint64_t)p;
    }
    if (!select(sg, kreq, j, a, s)) return kFail;
    if (CHK && L >= capL) return kENoMeta;
    if (CHK && L >= live_room) return kOverflow;
    if (s > sg) {  // Alg. 1 / Alg. 4: the block is cut from the low end
      if (CHK && kSeg && clock >= kStampLimit) return kOverflow;
      write<kAddr>(j, a + sg, 0u, kSeg ? seg_key(s - sg) : 0u);
    } else {
      remove<CHK>(j);
    }
    live_write(L, a, sg);
    ++L;
    if (ALGO == kNextFit) {
      rover = a + sg;
      hint = j;
    }
    return (int64_t)(uint64_t)a;
  }

  // Free live entry idx except its first floor(cut * size / 2^31) granules
  // (partial deallocation, sequential fits only; cut < 2^31): coalesce the
  // released part with free neighbours (Alg. 2 / Alg. 5), then shrink the
  // entry or, for a whole free, drop it from the live table (the last one
  // moves into its place).  Returns the first granule of the released part,
  // kENoMeta or kOverflow.
  template <bool CHK = true>
  __device__ __forceinline__ int64_t free_index(uint32_t idx, uint32_t cut) {
    if (CHK && kSeg && clock >= kStampLimit) return kOverflow;
    // The victim and the last live entry (which takes the victim's slot at
    // the end) are read together, so the second load's latency hides behind
    // the first; nothing below writes the live table before that move.
    const uint32_t lastL = L - 1u;
    uint32_t bx, bsz;
    wave_sync();
    const Ent victim = *live_ptr(idx), moved = *live_ptr(lastL);
    bx = uniform(ent_a(victim));
    bsz = uniform(ent_s(victim));
    const uint32_t t = (kSeg || cut == 0u) ? 0u : (uint32_t)(((uint64_t)cut * bsz) >> 31);
    const uint32_t x = bx + t, sz = bsz - t;  // the part released
    // A block ending at granule ~0 (an arena of 2^32 - 1 granules) has no
    // right neighbour; its own start, which no free block has, stands in for
    // its end so that empty slots (address ~0) do not match.
    const uint32_t end = x + sz, xe = end == kNone ? x : end;
    // chunk + 1 of this lane's left / right neighbour (0: none); there is at
    // most one of each, so two ballots after the scan find them
    uint32_t cl = 0, cr = 0;
    scan([&](uint32_t c, uint32_t ea, uint32_t ee, uint32_t) {
      cl = ee == x ? c + 1u : cl;
      cr = ea == xe ? c + 1u : cr;
    });
    const uint64_t ML = ballot(cl != 0u), MR = ballot(cr != 0u);
    if ((ML | MR) == 0ull) {
      if (CHK && F >= capF) return kENoMeta;
      // (the freed block still counts as live here: the check is on the safe side)
      if (CHK && need_bytes(F + 1u, L) > m.bytes) return kOverflow;
      append<CHK>(x, end, kSeg ? seg_key(sz) : 0u);
    } else if (MR == 0ull) {
      const uint32_t l = ctz64(ML), jl = 64u * (rdlane(cl, l) - 1u) + l;
      write<kEnd>(jl, 0u, end, kSeg ? seg_key(end - addr_at(jl)) : 0u);
    } else if (ML == 0ull) {
      const uint32_t l = ctz64(MR), jr = 64u * (rdlane(cr, l) - 1u) + l;
      write<kAddr>(jr, x, 0u, kSeg ? seg_key(end_at(jr) - x) : 0u);
    } else {
      // the left neighbour takes the merged block and the right one's entry
      // goes
      const uint32_t ll = ctz64(ML), jl = 64u * (rdlane(cl, ll) - 1u) + ll;
      const uint32_t lr = ctz64(MR), jr = 64u * (rdlane(cr, lr) - 1u) + lr;
      const uint32_t er = end_at(jr);
      write<kEnd>(jl, 0u, er, kSeg ? seg_key(er - addr_at(jl)) : 0u);
      remove<CHK>(jr);
    }
    if (t != 0u) {
      live_write(idx, bx, t);
    } else {
      wave_sync();
      *live_ptr(idx) = moved;  // idx == lastL rewrites the entry about to be dropped
      L = lastL;
    }
    return (int64_t)(uint64_t)x;
  }

  // Replay free: r is the 32-bit draw, the victim is live[(r * L) >> 32];
  // cut as in free_index; nothing live -> -1.
  template <bool CHK = true>
  __device__ __forceinline__ int64_t free_draw(uint32_t r, uint32_t cut) {
    if (CHK && L == 0u) return kFail;
    return free_index<CHK>((uint32_t)(((uint64_t)r * (uint64_t)L) >> 32), cut);
  }

  // Whether the next n (<= 64) requests can skip the overflow and capacity
  // checks: each adds at most one live entry and one free entry, n free
  // entries open at most one new LDS chunk (64 entries of kRec bytes, the
  // room of 8 kRec live entries), and each takes at most one push stamp;
  // with n live blocks to start from, no free finds the live table empty.
  __device__ __forceinline__ bool block_safe(uint32_t n) const {
    return L + n + 8u * kRec <= live_room && L + n <= capL && F + n <= capF && L >= n &&
           (!kSeg || clock + n < kStampLimit);
  }

  // Hand this heap over to the general core (hda_core.h) on tiers `c` with
  // no LDS part: every free entry i goes to device slot i with its push stamp
  // beside it, every live entry i to device slot i.
  __device__ void migrate(const Cold& c, HeapRegs& h) {
    const uint32_t lane = lane_id();
    const uint32_t counts = ALGO == kSegFit ? class_counts() : 0u;
    for (uint32_t ch = RF; 64u * ch < F; ++ch) {
      const uint32_t gi = 64u * ch + lane;
      wave_sync();
      uint32_t a, e, k;
      chunk_get(ch, a, e, k);
      if (gi < F) {
        c.gf[gi] = mk_ent(a, e - a);
        if (kSeg) c.gst[gi] = (k & kStampMask) ^ kStampMask;
      }
    }
#pragma unroll
    for (int k = 0; k < RF; ++k) {
      const uint32_t gi = 64u * (uint32_t)k + lane;
      if (gi < F) {
        c.gf[gi] = mk_ent(fa[k], fe[k] - fa[k]);
        if (kSeg) c.gst[gi] = (fk[k] & kStampMask) ^ kStampMask;
      }
    }
    for (uint32_t base = 0; base < L; base += 64u) {
      const uint32_t i = base + lane;
      wave_sync();
      const Ent e = *live_ptr(i < L ? i : 0u);
      if (i < L) c.gl[i] = e;
    }
    wave_sync();
    h.F = F;
    h.L = L;
    h.rover = rover;
    h.clock = clock;
    h.cnt = counts;
  }

  // Canonical state, same format as the general core (hda.h).
  __device__ int64_t dump(int64_t* out, int64_t cap) {
    const uint32_t lane = lane_id();
    const int64_t need = 4 + 2 * (int64_t)F + 2 * (int64_t)L + (kSeg ? kClasses + (int64_t)F : 0);
    if (out == nullptr || need > cap) return need;
    const uint32_t sh = shift;
    if (lane == 0) out[0] = F;
    int64_t* fo = out + 1;
    // free blocks ranked by address
    scan([&](uint32_t c, uint32_t a, uint32_t e, uint32_t) {
      const bool v = 64u * c + lane < F;
      uint32_t rank = 0;
      for (uint32_t j = 0; j < F; ++j) {
        uint32_t aj, sj, kj;
        read(j, aj, sj, kj);
        rank += aj < a ? 1u : 0u;
      }
      if (v) {
        fo[2 * rank] = (int64_t)((uint64_t)a << sh);
        fo[2 * rank + 1] = (int64_t)((uint64_t)(e - a) << sh);
      }
    });
    int64_t* lo = out + 1 + 2 * (int64_t)F;
    if (lane == 0) lo[0] = L;
    for (uint32_t base = 0; base < L; base += 64u) {
      const uint32_t i = base + lane;
      wave_sync();
      const Ent e = *live_ptr(i < L ? i : 0u);
      if (i < L) {
        lo[1 + 2 * i] = (int64_t)((uint64_t)ent_a(e) << sh);
        lo[2 + 2 * i] = (int64_t)((uint64_t)ent_s(e) << sh);
      }
    }
    int64_t* tail = lo + 1 + 2 * (int64_t)L;
    const uint32_t cnt = ALGO == kSegFit ? class_counts() : 0u;
    uint64_t bm = ballot(cnt != 0u);
    if constexpr (ALGO == kTlsf) {  // first level: the levels holding a free block
      bm = 0ull;
      for (uint32_t j = 0; j < F; ++j) {
        uint32_t aj, sj, kj;
        read(j, aj, sj, kj);
        bm |= 1ull << ((kj >> kKeyShift) / kNsl);
      }
    }
    if (lane == 0) {
      tail[0] = kRover ? (int64_t)((uint64_t)rover << sh) : -1;
      tail[1] = kSeg ? (int64_t)bm : 0;
    }
    if constexpr (ALGO == kTlsf) {
      // List c starts at word c + (free blocks in lower classes).  In key
      // order (by class, then last pushed first) a block is at word class +
      // 1 + its rank, and the word before a class's first block holds the
      // list's length; every other word is an empty list's 0.  One count over
      // the table per 64 blocks instead of one per 64 classes: 4,096 heaps x
      // 20,000 requests 10.6 -> 9.9 ms, state dumps included.
      int64_t* ls = tail + 2;
      const uint32_t words = kClasses + F;
      for (uint32_t i = lane; i < words; i += 64u) ls[i] = 0;
      stores_done();
      each_chunk([&](uint32_t c, uint32_t a, uint32_t, uint32_t key) {
        const bool v = 64u * c + lane < F;
        const uint32_t cls = key >> kKeyShift;
        uint32_t rank = 0, upto = 0;  // blocks before this one; in its class or before
        bool first = true;            // of its class
        for (uint32_t j = 0; j < F; ++j) {
          uint32_t aj, sj, kj;
          read(j, aj, sj, kj);
          const uint32_t cj = kj >> kKeyShift;
          rank += kj < key ? 1u : 0u;
          upto += cj <= cls ? 1u : 0u;
          first = first && !(cj == cls && kj < key);
        }
        if (v) ls[cls + 1u + rank] = (int64_t)((uint64_t)a << sh);
        if (v && first) ls[cls + rank] = (int64_t)(uint64_t)(upto - rank);
      });
    } else if constexpr (kSeg) {
      int64_t* ls = tail + 2;
      const uint32_t region = 64u + F;  // words of the class-list section
      // header position of class `lane`: sum over lower classes of (1 + count)
      uint32_t hdr = 0, acc = 0;
      for (uint32_t k = 0; k < 64u; ++k) {
        hdr = (lane == k) ? acc : hdr;
        acc += 1u + rdlane(cnt, k);
      }
      if (hdr < region) ls[hdr] = cnt;
      // within a class, blocks from the last pushed (smallest key) on
      scan([&](uint32_t c, uint32_t a, uint32_t, uint32_t key) {
        const bool v = 64u * c + lane < F;
        const uint32_t cls = v ? key >> kKeyShift : 0u;
        uint32_t rank = 0;
        for (uint32_t j = 0; j < F; ++j) {
          uint32_t aj, sj, kj;
          read(j, aj, sj, kj);
          rank += ((kj >> kKeyShift) == cls && kj < key) ? 1u : 0u;
        }
        const uint32_t hc = shfl(hdr, cls);
        if (v && hc + 1u + rank < region) ls[hc + 1u + rank] = (int64_t)((uint64_t)a << sh);
      });
    }
    return need;
  }
};

}  // namespace hda
