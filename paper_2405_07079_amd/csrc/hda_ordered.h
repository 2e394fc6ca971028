// Ordered replay core: one wavefront replays one heap with its free blocks
// kept in address order, so that every step of Alg. 1-5 costs a fixed number
// of wave operations however many free blocks the heap has.
//
// Free blocks form a sorted array of 64-entry chunks, one entry per lane --
// the hybrid array list of App. A, whose traversal costs O(n/m + m) on one
// CPU thread.  Here a directory held in D VGPRs replaces the walk over the
// chunk list: lane l of directory register v describes chunk 64 v + l in
// order (its storage slot, its number of entries, its first key and, for
// first and next fit, the largest block in it).  Finding the chunk that
// holds a key, or the first chunk holding a block of at least s granules,
// is one ballot per directory register; finding the entry inside it is one
// chunk load and one ballot.  A full chunk splits into 33 + 32 entries; a
// chunk that drops below 32 entries merges with a neighbour or takes entries
// from it.  So while there are two or more chunks each holds at least 32
// entries, and the directory's 64 D chunks always hold 2,048 D free blocks.
//
// A free block's entry is keyed by its LAST granule.  Free blocks do not
// overlap, so this is also address order, and Alg. 1 / Alg. 4 cut an
// allocation from the low end of a block: the remainder keeps its end, so
// splitting a block rewrites its size (or its record) and never its place.
// The block ending right below a freed block's start is an exact key match;
// the one after it is the next entry.  No block's last granule is kNone
// (arenas end at 2^32 - 1 granules), so kNone fills the unused entries and
// directory lanes and every search is one strict comparison with no mask:
// "last granule < x" is "end <= x".
//
// Per algorithm:
//  * first fit (Sec. II-A): entries (last granule, size); the first chunk whose
//    largest block fits, then the first fitting entry in it.
//  * next fit (Sec. II-A, Sec. IV): the first block ending past the rover
//    is located like a key; the search runs on from there through the
//    directory and wraps once.
//  * best fit (Alg. 3): entries (last granule, size) and a second sorted
//    chunk table of keys (size, last granule) -- among blocks of one size the
//    lowest is the lowest address; the smallest key at or above (s, 0) is the best fit.
//  * segregated fit (Alg. 4-5) and TLSF (Sec. V-B): entries (last granule,
//    record).
//    A record holds the block's address and size and its class-list links
//    (next and previous record, NIL = kNone), as Alg. 4-5 keep them; record
//    numbers never change while a block is free, so unlinking and pushing
//    are stores with no search.  Free record numbers are bits of a VGPR
//    pair (lane l: records 64 l .. 64 l + 63).  List heads are in a VGPR
//    (segregated fit: lane k heads class k) or in LDS (TLSF's 2,048
//    classes); the bitmaps are a scalar (segregated fit; TLSF's first level)
//    and a VGPR (TLSF's second level: lane fl holds level fl's 32 bits).
//    The paper's address-keyed hash lookup ht[addr] becomes the key lookup
//    in the table.
//
// What bounds it: one wave alone issues an instruction every four clocks and
// waits about 130 for each dependent LDS read, and no other wave hides that.
// So searches take no masks, a chunk's largest block is reduced anew only
// when that block goes, the record given back last is taken next, the next
// free's victim is loaded while the current request runs, and the LDS side of
// every access falls through.  First 100,000-300,000 requests of the 256 GiB
// traces, per request: first fit 466 -> 396 ns, next fit 521 -> 435, best fit
// 722 -> 652, segregated fit 657 -> 617, TLSF 815 -> 733.  (Tried and not
// kept: best fit's remainder chunk loaded before the old key is removed, 2 %
// slower; writing a chunk's first key only when it changes, 2-4 % slower.)
//
// Results equal those of the other cores and the oracle: selection,
// splitting, merging and the class lists follow the same definitions.
//
// Storage: chunk slots, records and live entries below the LDS counts given
// at construction are in the wave's LDS pool, the rest in its device-memory
// slot.  Every memory access is preceded by wave_sync() (a no-op on the GPU;
// the CPU wave emulation switches lanes there).  As in the other cores,
// values that feed a cross-lane operation are never produced under a
// lane-dependent branch, and every single-entry write is done by all lanes
// with the same value.
#pragma once
#include <stdint.h>

#include "hda_core.h"

namespace hda {

// 8- and 16-byte entries as plain vectors (loaded and stored whole through
// pointers of any address space).
typedef uint32_t u32x2 __attribute__((vector_size(8)));
typedef uint32_t u32x4 __attribute__((vector_size(16)));

// A branch whose other side is out of the way: a lone wave pays a taken
// branch with an instruction fetch, so the LDS side of a table access and
// the common outcomes fall through.
__device__ __forceinline__ bool likely(bool c) { return __builtin_expect(c, true); }
__device__ __forceinline__ bool unlikely(bool c) { return __builtin_expect(c, false); }

// Wave-wide maximum of a u32 (every lane active).
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return ~wave_min(~v); }

// The lanes below n as a mask (n <= 64 or more): lane conditions of a ballot
// are applied on the scalar side instead of being combined per lane.
__device__ __forceinline__ uint64_t lanes_below(uint32_t n) {
  return n >= 64u ? ~0ull : (1ull << n) - 1ull;
}

// Memory accesses before this point are not moved past it by the compiler
// (the hardware keeps a wave's accesses in order): for data that one lane
// writes and another reads.
__device__ __forceinline__ void wave_order() {
  wave_sync();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Directory access: lane (i & 63) of register i >> 6.
template <int D>
__device__ __forceinline__ uint32_t dir_get(const uint32_t (&v)[D], uint32_t i) {
  uint32_t x = rdlane(v[0], i & 63u);
#pragma unroll
  for (int k = 1; k < D; ++k) {
    const uint32_t y = rdlane(v[k], i & 63u);
    x = (i >> 6) == (uint32_t)k ? y : x;
  }
  return x;
}
template <int D>
__device__ __forceinline__ void dir_put(uint32_t (&v)[D], uint32_t i, uint32_t x) {
  if constexpr (D == 1) {
    v[0] = put_lane(v[0], i, x);
  } else {
    const bool me = lane_id() == (i & 63u);
#pragma unroll
    for (int k = 0; k < D; ++k) v[k] = (me && (i >> 6) == (uint32_t)k) ? x : v[k];
  }
}
// Open a hole at directory position i (entries i.. move up by one; the last
// one falls off) and put x there.
template <int D>
__device__ __forceinline__ void dir_insert(uint32_t (&v)[D], uint32_t i, uint32_t x) {
  const uint32_t lane = lane_id();
  uint32_t carry = x;  // lane 63 of the register below, before the shift
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint32_t top = rdlane(v[k], 63);
    const uint32_t moved = wave_shr1(carry, v[k]);  // lane 0 takes the carry
    const uint32_t g = 64u * (uint32_t)k + lane;
    v[k] = g > i ? moved : (g == i ? x : v[k]);
    carry = top;
  }
}
// Remove directory position i (entries past it move down); the last
// position receives `fill`.
template <int D>
__device__ __forceinline__ void dir_erase(uint32_t (&v)[D], uint32_t i, uint32_t fill) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint32_t next0 = k + 1 < D ? rdlane(v[k + 1 < D ? k + 1 : k], 0) : fill;
    const uint32_t moved = wave_shl1(next0, v[k]);  // lane 63 takes the next register's lane 0
    const uint32_t g = 64u * (uint32_t)k + lane;
    v[k] = g >= i ? moved : v[k];
  }
}

// One table of sorted chunks of 8-byte entries (key, value): the key is a
// block's last granule, the value its size or its record.  KEY64: sorted by
// (value, key) instead (best fit's keys).  MAXS: the directory
// keeps each chunk's largest value (first and next fit: the largest size).
template <bool KEY64, bool MAXS, int D>
struct Hal {
  static constexpr uint32_t NC = 64u * D;  // chunk slots
  static constexpr uint32_t CB = 64u * 8u; // bytes per chunk

  // this lane's entry of a loaded chunk; positions past the chunk's count
  // hold the sentinel (key kNone, value 0, or value kNone when sorted by
  // value), which sorts after every real entry and fits no request
  struct Row {
    uint32_t a, s;
  };

  static constexpr int ND = D;
  HDA_LDS uint8_t* lb;     // slots [0, nl) in LDS
  HDA_GLOBAL uint8_t* gb;  // slot i >= nl at gb + i * CB in device memory
  uint32_t nl, nl_req;     // LDS slots (nl_req as asked for, nl within NC)
  uint32_t dsl[D], dct[D], dk0[D], dk1[D], dmx[D];  // slot, count, first key, max value
  uint64_t used[D];                                 // slots in use
  uint32_t nc;                                      // chunks

  static constexpr uint32_t kSentS = KEY64 ? kNone : 0u;

  __device__ __forceinline__ static Row sentinel() { return Row{kNone, kSentS}; }

  __device__ __forceinline__ void init(HDA_LDS uint8_t* l, HDA_GLOBAL uint8_t* g, uint32_t n_lds) {
    lb = l;
    gb = g;
    nl_req = n_lds;
    nl = n_lds < NC ? n_lds : NC;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      dsl[k] = 0u; dct[k] = 0u; dk0[k] = kNone; dk1[k] = kNone; dmx[k] = 0u;
      used[k] = 0ull;
    }
    nc = 0;
  }

  // ---- chunk memory (slot ids are below NC; the clamps keep every access
  // inside the table whatever happens) ----
  __device__ __forceinline__ Row load(uint32_t sl) const {
    wave_sync();
    sl = sl < NC ? sl : NC - 1u;
    const uint32_t lane = lane_id();
    u32x2 v;
    if (likely(sl < nl)) {
      v = *(const HDA_LDS u32x2*)(lb + sl * CB + lane * 8u);
    } else {
      v = *(const HDA_GLOBAL u32x2*)(gb + (uint64_t)sl * CB + lane * 8u);
      settle(v[0]);
      settle(v[1]);
    }
    return Row{v[0], v[1]};
  }
  __device__ __forceinline__ void store(uint32_t sl, const Row& r) const {
    wave_sync();
    sl = sl < NC ? sl : NC - 1u;
    const uint32_t lane = lane_id();
    u32x2 v;
    v[0] = r.a; v[1] = r.s;
    if (likely(sl < nl)) *(HDA_LDS u32x2*)(lb + sl * CB + lane * 8u) = v;
    else *(HDA_GLOBAL u32x2*)(gb + (uint64_t)sl * CB + lane * 8u) = v;
  }
  // field f (0 key, 1 value) of entry p, written by every lane
  __device__ __forceinline__ void store_field(uint32_t sl, uint32_t p, uint32_t f,
                                              uint32_t x) const {
    wave_sync();
    sl = sl < NC ? sl : NC - 1u;
    const uint32_t off = (p & 63u) * 8u + (f & 1u) * 4u;
    if (likely(sl < nl)) *(HDA_LDS uint32_t*)(lb + sl * CB + off) = x;
    else *(HDA_GLOBAL uint32_t*)(gb + (uint64_t)sl * CB + off) = x;
  }
  __device__ __forceinline__ void store_entry(uint32_t sl, uint32_t p, uint32_t a,
                                              uint32_t s) const {
    wave_sync();
    sl = sl < NC ? sl : NC - 1u;
    u32x2 v;
    v[0] = a; v[1] = s;
    const uint32_t off = (p & 63u) * 8u;
    if (likely(sl < nl)) *(HDA_LDS u32x2*)(lb + sl * CB + off) = v;
    else *(HDA_GLOBAL u32x2*)(gb + (uint64_t)sl * CB + off) = v;
  }

  // ---- keys ----
  // Lanes whose key (r1, r0) is below (k1, k0); keyed by r0 alone unless
  // KEY64 (then as one 64-bit value: one vector compare).
  __device__ __forceinline__ static uint64_t key_ballot(uint32_t r1, uint32_t r0, uint32_t k1,
                                                        uint32_t k0) {
    if constexpr (!KEY64) return ballot(r0 < k0);
    return ballot((((uint64_t)r1 << 32) | r0) < (((uint64_t)k1 << 32) | k0));
  }
  // chunks whose first key is below (k1, k0)
  __device__ __forceinline__ uint32_t count_first(uint32_t k1, uint32_t k0) const {
    uint32_t n = 0;
#pragma unroll
    for (int k = 0; k < D; ++k)
      n += (uint32_t)__builtin_popcountll(key_ballot(dk1[k], dk0[k], k1, k0));
    return n;
  }

  __device__ __forceinline__ uint32_t slot(uint32_t ci) const { return dir_get(dsl, ci); }
  __device__ __forceinline__ uint32_t count(uint32_t ci) const { return dir_get(dct, ci); }

  // Directory entry of chunk ci from its row (n entries).
  __device__ __forceinline__ void describe(uint32_t ci, const Row& r, uint32_t n) {
    dir_put(dct, ci, n);
    dir_put(dk0, ci, rdlane(r.a, 0));
    if (KEY64) dir_put(dk1, ci, rdlane(r.s, 0));
    if (MAXS) dir_put(dmx, ci, wave_max(r.s));
  }

  // the entry chunk ci starts with (written whether it changed or not: a
  // test costs as much and a branch more)
  __device__ __forceinline__ void first(uint32_t ci, uint32_t a, uint32_t s) {
    dir_put(dk0, ci, a);
    if (KEY64) dir_put(dk1, ci, s);
  }
  // A chunk's largest value when one of them has grown to s, or when one
  // that was s is gone or smaller (row o is what is left): only the largest
  // itself going takes a reduction over the row.
  __device__ __forceinline__ void grow(uint32_t ci, uint32_t s) {
    const uint32_t old = dir_get(dmx, ci);
    dir_put(dmx, ci, old > s ? old : s);
  }
  __device__ __forceinline__ void shrink(uint32_t ci, uint32_t s, const Row& o) {
    if (unlikely(s == dir_get(dmx, ci))) dir_put(dmx, ci, wave_max(o.s));
  }

  __device__ __forceinline__ uint32_t take_slot() {
    uint32_t s = kNone;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      const uint64_t fr = ~used[k];
      s = fr != 0ull ? 64u * (uint32_t)k + ctz64(fr) : s;
    }
    // the occupancy rule leaves a free slot whenever a chunk is added; the
    // last slot stands in should that ever fail, so no access leaves the table
    s = s == kNone ? NC - 1u : s;
#pragma unroll
    for (int k = 0; k < D; ++k)
      used[k] |= (s >> 6) == (uint32_t)k ? 1ull << (s & 63u) : 0ull;
    return s;
  }
  __device__ __forceinline__ void drop_slot(uint32_t s) {
#pragma unroll
    for (int k = 0; k < D; ++k)
      used[k] &= (s >> 6) == (uint32_t)k ? ~(1ull << (s & 63u)) : ~0ull;
  }

  // A table holding one entry.
  __device__ __forceinline__ void start(uint32_t a, uint32_t s) {
    const uint32_t sl = take_slot();
    Row r = sentinel();
    const bool me = lane_id() == 0u;
    r.a = me ? a : r.a;
    r.s = me ? s : r.s;
    store(sl, r);
    nc = 1;
    dir_put(dsl, 0u, sl);
    describe(0u, r, 1u);
  }

  // Row shifted: lane l receives lane src(l) of r (the sentinel when !ok).
  __device__ __forceinline__ static Row pull(const Row& r, uint32_t src, bool ok) {
    const uint32_t s = src & 63u;
    Row o{shfl(r.a, s), shfl(r.s, s)};
    o.a = ok ? o.a : kNone;
    o.s = ok ? o.s : kSentS;
    return o;
  }
  __device__ __forceinline__ static Row pick(bool c, const Row& x, const Row& y) {
    return Row{c ? x.a : y.a, c ? x.s : y.s};
  }
  // r with lane p's entry replaced
  __device__ __forceinline__ static Row with(const Row& r, uint32_t p, uint32_t a, uint32_t s) {
    const bool me = lane_id() == p;
    return Row{me ? a : r.a, me ? s : r.s};
  }

  // Insert entry e at position p (0 <= p <= count) of chunk ci, whose row r
  // is current.  The caller guarantees order and capacity.
  __device__ __forceinline__ void insert_at(uint32_t ci, uint32_t p, const Row& r, const Row& e) {
    const uint32_t lane = lane_id();
    const uint32_t n = count(ci), sl = slot(ci);
    // the row moved up one lane (lane 0: the sentinel)
    const Row up{wave_shr1(kNone, r.a), wave_shr1(kSentS, r.s)};
    if (likely(n < 64u)) {
      const Row o = pick(lane < p, r, pick(lane == p, e, up));
      store(sl, o);
      dir_put(dct, ci, n + 1u);
      first(ci, rdlane(o.a, 0), KEY64 ? rdlane(o.s, 0) : 0u);
      if (MAXS) grow(ci, e.s);
      return;
    }
    // split: the 65 entries c[0..64] become 33 here and 32 in a new chunk
    // after it; c[i] = r[i] (i < p), e (i == p), r[i - 1] (i > p)
    const uint32_t ns = take_slot();
    Row left = pick(lane < p, r, pick(lane == p, e, up));
    left = pick(lane <= 32u, left, sentinel());
    const uint32_t i = lane + 33u;  // position in c of this lane's right entry
    const Row r_same = pull(r, i, i < 64u);
    const Row r_prev = pull(r, i - 1u, true);
    Row right = pick(i < p, r_same, pick(i == p, e, r_prev));
    right = pick(lane < 32u, right, sentinel());
    store(sl, left);
    store(ns, right);
    describe(ci, left, 33u);
    dir_insert(dsl, ci + 1u, ns);
    dir_insert(dct, ci + 1u, 32u);
    dir_insert(dk0, ci + 1u, rdlane(right.a, 0));
    if (KEY64) dir_insert(dk1, ci + 1u, rdlane(right.s, 0));
    if (MAXS) dir_insert(dmx, ci + 1u, wave_max(right.s));
    ++nc;
  }

  // Remove the entry at position p of chunk ci (row r current), then keep
  // every chunk at 32 entries or more while there are two or more.
  __device__ __forceinline__ void erase_at(uint32_t ci, uint32_t p, const Row& r) {
    const uint32_t lane = lane_id();
    const uint32_t n = count(ci) - 1u, sl = slot(ci);
    // the row moved down one lane (lane 63: the sentinel)
    const Row down{wave_shl1(kNone, r.a), wave_shl1(kSentS, r.s)};
    const Row o = pick(lane >= p, down, r);
    if (likely(n >= 32u || nc == 1u)) {
      store(sl, o);
      dir_put(dct, ci, n);
      first(ci, rdlane(o.a, 0), KEY64 ? rdlane(o.s, 0) : 0u);
      if (MAXS) shrink(ci, rdlane(r.s, p), o);
      return;
    }
    // join with the next chunk (or the previous one for the last chunk)
    const uint32_t lo = ci + 1u < nc ? ci : ci - 1u, hi = lo + 1u;
    const uint32_t sl_lo = slot(lo), sl_hi = slot(hi);
    const Row other = load(ci == lo ? sl_hi : sl_lo);
    const Row L = ci == lo ? o : other, H = ci == lo ? other : o;
    const uint32_t nL = ci == lo ? n : count(lo), nH = ci == lo ? count(hi) : n;
    const uint32_t T = nL + nH;
    // c[i] = L[i] (i < nL), H[i - nL] (i >= nL)
    if (T <= 64u) {
      const Row hp = pull(H, lane - nL, lane >= nL && lane < T);
      const Row m = pick(lane < nL, L, hp);
      store(sl_lo, m);
      describe(lo, m, T);
      drop_slot(sl_hi);
      dir_erase(dsl, hi, 0u);
      dir_erase(dct, hi, 0u);
      dir_erase(dk0, hi, kNone);
      if (KEY64) dir_erase(dk1, hi, kNone);
      if (MAXS) dir_erase(dmx, hi, 0u);
      --nc;
      return;
    }
    // share the T (65..95) entries: T / 2 in the lower chunk, the rest above
    const uint32_t a = T >> 1, b = T - a;
    const Row hp = pull(H, lane - nL, lane >= nL);
    Row m0 = pick(lane < nL, L, hp);
    m0 = pick(lane < a, m0, sentinel());
    const uint32_t i = lane + a;
    const Row lsrc = pull(L, i, i < nL);
    const Row hsrc = pull(H, i - nL, i >= nL && i < T);
    Row m1 = pick(i < nL, lsrc, hsrc);
    m1 = pick(lane < b, m1, sentinel());
    store(sl_lo, m0);
    store(sl_hi, m1);
    describe(lo, m0, a);
    describe(hi, m1, b);
  }

  // Where key (k1, k0) belongs: chunk ci (the last one starting below it,
  // else the first), its row, and the number q of its entries below the key.
  // An entry equal to the key is at position q, or starts the next chunk; to
  // find it, ask for the key one above it: it is then at q - 1.
  __device__ __forceinline__ void locate(uint32_t k1, uint32_t k0, uint32_t& ci, Row& r,
                                         uint32_t& q) const {
    const uint32_t c = count_first(k1, k0);
    ci = c != 0u ? c - 1u : 0u;
    r = load(slot(ci));
    q = (uint32_t)__builtin_popcountll(key_ballot(r.s, r.a, k1, k0));
  }
  // (value, key) tables: insert and remove one key
  __device__ __forceinline__ void insert_key(uint32_t a, uint32_t s) {
    uint32_t ci, q;
    Row r;
    locate(s, a, ci, r, q);
    insert_at(ci, q, r, Row{a, s});
  }
  __device__ __forceinline__ void erase_key(uint32_t a, uint32_t s) {
    uint32_t ci, q;
    Row r;
    locate(s, a + 1u, ci, r, q);
    erase_at(ci, q - 1u, r);
  }
  // first chunk at or after `from` whose largest value is >= sg (MAXS
  // tables), or kNone
  __device__ __forceinline__ uint32_t first_fit_chunk(uint32_t sg, uint32_t from) const {
    uint32_t c = kNone;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      const uint32_t base = 64u * (uint32_t)k;  // (unused lanes hold 0)
      const uint64_t m = ballot(dmx[k] >= sg) & ~lanes_below(from > base ? from - base : 0u);
      c = m != 0ull ? 64u * (uint32_t)k + ctz64(m) : c;
    }
    return c;
  }
};

// Where one heap's tables live.  Table slots, records and live entries below
// the LDS counts are in the wave's LDS pool; the others are in its device
// slot.
struct OrdMem {
  HDA_LDS uint8_t* ta_l;
  HDA_GLOBAL uint8_t* ta_g;
  uint32_t ta_n;
  HDA_LDS uint8_t* tb_l;     // best fit's key table
  HDA_GLOBAL uint8_t* tb_g;
  uint32_t tb_n;
  HDA_LDS u32x4* rec_l;      // segregated fit / TLSF records
  HDA_GLOBAL u32x4* rec_g;
  uint32_t rec_n;
  HDA_LDS Ent* ll;
  HDA_GLOBAL Ent* gl;
  uint32_t ll_n;
  HDA_LDS uint32_t* heads;   // TLSF list heads (2,048 words, LDS)
};

constexpr int kOrdDir = 2;                          // directory registers at most
constexpr uint32_t kOrdSlots = 64u * kOrdDir;      // chunk slots per table
constexpr uint32_t kOrdMaxFree = 32u * kOrdSlots;  // free blocks always held
constexpr uint32_t kOrdTlsfHeadBytes = kTlsfClasses * 4u;
constexpr uint32_t kOrdChunkBytes = 64u * 8u;
// Device bytes per wave: every chunk slot of the table (64 KiB), then best
// fit's key table or the records (64 KiB either), then the live table.
// Slots, records and entries held in LDS keep an unused place here.
constexpr uint64_t kOrdTableBytes = (uint64_t)kOrdSlots * kOrdChunkBytes;
constexpr uint64_t kOrdSecondBytes = (uint64_t)kOrdMaxFree * 16u;
static_assert(kOrdSecondBytes == kOrdTableBytes, "key table and records share one area");
__host__ __device__ constexpr uint64_t ord_dev_bytes(uint32_t cap_live) {
  return kOrdTableBytes + kOrdSecondBytes + (uint64_t)cap_live * 8u;
}

// A heap that starts on the lean core and moves here (OrdHeap::adopt) has a
// device slot cut to its capacity: chunks hold at least 32 entries, so
// cap_free entries (a multiple of 64) take at most cap_free / 32 chunk slots,
// 16 bytes an entry, and its records or key table the same.
__host__ __device__ constexpr uint64_t ord_area_bytes(uint32_t cap_free) {
  return (uint64_t)cap_free * 16u;
}
__host__ __device__ constexpr uint64_t ord_spill_bytes(uint32_t cap_free, uint32_t cap_live) {
  return 2u * ord_area_bytes(cap_free) + (uint64_t)cap_live * 8u;
}
// Free blocks such a heap may bring: adopt() stages them beside the chunks
// (9.2 bytes an entry) and beside the records (16) it builds from them.
__host__ __device__ constexpr uint32_t ord_adopt_max(uint32_t cap_free) {
  return cap_free - cap_free / 4u;
}
// The least pool for it: TLSF's list heads are always in LDS.
constexpr uint32_t kOrdMinPool = kOrdTlsfHeadBytes + 2048u;

// Split a wave's pool (`pool_bytes`, of which `slot_bytes` are meant for the
// tables and records) and its device slot, whose two table areas take
// `area_bytes` each, for an algorithm.
__device__ __forceinline__ OrdMem ord_mem(int algo, HDA_LDS uint8_t* pool, uint32_t pool_bytes,
                                          uint32_t slot_bytes, HDA_GLOBAL uint8_t* dev,
                                          uint32_t cap_live,
                                          uint32_t area_bytes = (uint32_t)kOrdTableBytes) {
  OrdMem m;
  uint32_t off = 0;
  m.heads = (HDA_LDS uint32_t*)pool;
  if (algo == kTlsf) off += kOrdTlsfHeadBytes;
  const uint32_t room = pool_bytes > off ? pool_bytes - off : 0u;
  const uint32_t area = slot_bytes < room ? slot_bytes : room;
  // first and next fit: every slot of the table; best fit: half for each of
  // its two tables; segregated fit, TLSF: half for table slots, half for
  // records
  const bool two = algo == kBestFit || seg_like(algo);
  uint32_t na = (two ? area / 2u : area) / kOrdChunkBytes;
  na = na < kOrdSlots ? na : kOrdSlots;
  m.ta_l = pool + off;
  m.ta_n = na;
  off += na * kOrdChunkBytes;
  m.tb_l = pool + off;
  m.tb_n = algo == kBestFit ? na : 0u;
  off += algo == kBestFit ? na * kOrdChunkBytes : 0u;
  uint32_t nr = seg_like(algo) ? (area / 2u) / 16u : 0u;
  nr = nr < kOrdMaxFree ? nr : kOrdMaxFree;
  m.rec_l = (HDA_LDS u32x4*)(pool + off);
  m.rec_n = nr;
  off += nr * 16u;
  m.ta_g = dev;
  m.tb_g = dev + area_bytes;
  m.rec_g = (HDA_GLOBAL u32x4*)(dev + area_bytes);
  m.ll = (HDA_LDS Ent*)(pool + off);
  // whole 64-entry chunks, so that each lies on one side
  const uint32_t nl = pool_bytes > off ? ((pool_bytes - off) / 8u) & ~63u : 0u;
  m.ll_n = nl < cap_live ? nl : cap_live;
  m.gl = (HDA_GLOBAL Ent*)(dev + 2u * (uint64_t)area_bytes);
  return m;
}

// D: directory registers.  A heap starts with one; a request that finds a
// table at 64 chunks returns kOverflow before changing anything, and the
// heap continues with two (take()), which hold every table this core allows.
template <int ALGO, int D>
struct OrdHeap {
  static constexpr bool kSeg = ALGO == kSegFit || ALGO == kTlsf;
  static constexpr bool kKeys = ALGO == kBestFit;
  static constexpr bool kMax = ALGO == kFirstFit || ALGO == kNextFit;
  using TA = Hal<false, kMax, D>;
  using TB = Hal<true, false, D>;
  using Row = typename TA::Row;
  static constexpr bool kGranules = true;  // alloc / free_draw return granules

  TA ta;
  TB tb;
  OrdMem m;
  int64_t arena;
  uint32_t shift, ag;
  uint32_t F, L, rover;
  uint32_t capF, capL;
  uint32_t hd;          // segregated fit: lane k = head record of class k (kNone: empty)
  uint64_t bm;          // segregated fit: class bitmap; TLSF: first-level bitmap
  uint32_t slb;         // TLSF: lane fl = bitmap of the 32 sub-classes of level fl
  uint32_t frl, frh;    // free records: lane l, bit b <=> record 64 l + b (low, high word)
  uint32_t spare;       // one more free record, or kNone

  __device__ __forceinline__ OrdHeap(const OrdMem& mem, const HeapRegs& h, uint32_t cap_free,
                                     uint32_t cap_live)
      : m(mem), arena(h.arena), shift(h.shift), ag(h.ag),
        capF(cap_free < kOrdMaxFree ? cap_free : kOrdMaxFree), capL(cap_live) {}

  // ---- live table ----
  // (every lane reads the same entry)
  __device__ __forceinline__ Ent lraw(uint32_t i) const {
    wave_sync();
    if (likely(i < m.ll_n)) return m.ll[i];
    const Ent e = m.gl[i];
    settle((uint32_t)e);
    settle((uint32_t)(e >> 32));
    return e;
  }
  __device__ __forceinline__ void lset(uint32_t i, Ent e) const {
    wave_sync();
    if (likely(i < m.ll_n)) m.ll[i] = e; else m.gl[i] = e;  // every lane, same value
  }
  __device__ __forceinline__ Ent lchunk(uint32_t base) const {  // base: multiple of 64
    wave_sync();
    const uint32_t i = base + lane_id();
    if (base < m.ll_n) return m.ll[i];
    return m.gl[i];
  }

  // ---- records (segregated fit, TLSF): address, size, next, prev ----
  struct Rec {
    uint32_t a, s, nx, pv;
  };
  __device__ __forceinline__ u32x4 rec_raw(uint32_t i) const {
    wave_sync();
    i = i < kOrdMaxFree ? i : kOrdMaxFree - 1u;
    u32x4 v;
    if (likely(i < m.rec_n)) {
      v = m.rec_l[i];
    } else {
      v = m.rec_g[i];
      settle(v[0]); settle(v[1]); settle(v[2]); settle(v[3]);
    }
    return v;
  }
  __device__ __forceinline__ static Rec rec_of(const u32x4& v) {
    return Rec{uniform(v[0]), uniform(v[1]), uniform(v[2]), uniform(v[3])};
  }
  __device__ __forceinline__ Rec rec(uint32_t i) const { return rec_of(rec_raw(i)); }
  __device__ __forceinline__ void rec_put(uint32_t i, uint32_t a, uint32_t s, uint32_t nx,
                                          uint32_t pv) const {
    wave_sync();
    i = i < kOrdMaxFree ? i : kOrdMaxFree - 1u;
    u32x4 v;
    v[0] = a; v[1] = s; v[2] = nx; v[3] = pv;
    if (likely(i < m.rec_n)) m.rec_l[i] = v; else m.rec_g[i] = v;
  }
  // one field (2 next, 3 prev) of record i
  __device__ __forceinline__ void rec_link(uint32_t i, uint32_t f, uint32_t x) const {
    wave_sync();
    i = i < kOrdMaxFree ? i : kOrdMaxFree - 1u;
    if (likely(i < m.rec_n)) ((HDA_LDS uint32_t*)(m.rec_l + i))[f & 3u] = x;
    else ((HDA_GLOBAL uint32_t*)(m.rec_g + i))[f & 3u] = x;
  }
  // (the record given back last is taken first: spare)
  __device__ __forceinline__ uint32_t rec_take() {
    const uint32_t top = spare;
    if (likely(top != kNone)) {
      spare = kNone;
      return top;
    }
    const uint64_t m1 = ballot((frl | frh) != 0u);
    const uint32_t l = m1 != 0ull ? ctz64(m1) : 63u;
    const uint32_t wl = rdlane(frl, l), wh = rdlane(frh, l);
    const uint32_t b = wl != 0u ? (uint32_t)__builtin_ctz(wl)
                                : 32u + (uint32_t)__builtin_ctz(wh != 0u ? wh : 1u);
    const bool me = lane_id() == l;
    frl = me && b < 32u ? frl & ~(1u << b) : frl;
    frh = me && b >= 32u ? frh & ~(1u << (b - 32u)) : frh;
    return 64u * l + b;
  }
  __device__ __forceinline__ void rec_give(uint32_t i) {
    const uint32_t old = spare;
    spare = i;
    if (likely(old == kNone)) return;
    i = old;
    const bool me = lane_id() == (i >> 6);
    const uint32_t b = i & 63u;
    frl = me && b < 32u ? frl | (1u << b) : frl;
    frh = me && b >= 32u ? frh | (1u << (b - 32u)) : frh;
  }

  // ---- class lists (segregated fit, TLSF) ----
  __device__ __forceinline__ uint32_t cls(uint32_t sg) const {
    return ALGO == kTlsf ? tlsf_class(sg, shift) : floor_log2_u32(sg) + shift;
  }
  __device__ __forceinline__ uint32_t head(uint32_t c) const {
    if constexpr (ALGO == kTlsf) {
      wave_sync();
      return uniform(m.heads[c]);
    } else {
      return rdlane(hd, c);
    }
  }
  __device__ __forceinline__ void set_head(uint32_t c, uint32_t i) {
    if constexpr (ALGO == kTlsf) {
      wave_sync();
      m.heads[c] = i;
    } else {
      hd = put_lane(hd, c, i);
    }
  }
  __device__ __forceinline__ void bit_set(uint32_t c) {
    if constexpr (ALGO == kTlsf) {
      slb = put_lane(slb, c >> 5, rdlane(slb, c >> 5) | (1u << (c & 31u)));
      bm |= 1ull << (c >> 5);
    } else {
      bm |= 1ull << c;
    }
  }
  __device__ __forceinline__ void bit_clear(uint32_t c) {
    if constexpr (ALGO == kTlsf) {
      const uint32_t w = rdlane(slb, c >> 5) & ~(1u << (c & 31u));
      slb = put_lane(slb, c >> 5, w);
      bm &= w == 0u ? ~(1ull << (c >> 5)) : ~0ull;
    } else {
      bm &= ~(1ull << c);
    }
  }
  // Unlink a block of sg granules with links (nx, pv) from its class list.
  __device__ __forceinline__ void unlink(uint32_t sg, uint32_t nx, uint32_t pv) {
    const uint32_t c = cls(sg);
    if (pv == kNone) {
      set_head(c, nx);
      if (nx == kNone) bit_clear(c);
    } else {
      rec_link(pv, 2u, nx);
    }
    if (nx != kNone) rec_link(nx, 3u, pv);
  }
  // Record i becomes the head of its class list (Alg. 4-5 push) with block
  // (a, sg).
  __device__ __forceinline__ void push(uint32_t i, uint32_t a, uint32_t sg) {
    const uint32_t c = cls(sg);
    const uint32_t oh = head(c);
    if (oh != kNone) rec_link(oh, 3u, i);
    rec_put(i, a, sg, oh, kNone);
    set_head(c, i);
    bit_set(c);
  }

  // Alg. 6: one free block [0, A).
  __device__ __forceinline__ void init() {
    ta.init(m.ta_l, m.ta_g, m.ta_n);
    F = 1; L = 0; rover = 0;
    hd = kNone; bm = 0ull; slb = 0u; spare = kNone;
    if constexpr (kSeg) {
      // records 0 .. capF - 1 are free, then record 0 takes the arena
      const uint32_t base = 64u * lane_id();
      frl = base >= capF ? 0u : (capF - base >= 32u ? ~0u : (1u << (capF - base)) - 1u);
      frh = base + 32u >= capF ? 0u
            : (capF - base - 32u >= 32u ? ~0u : (1u << (capF - base - 32u)) - 1u);
      if constexpr (ALGO == kTlsf) {
        for (uint32_t c = 0; c < kTlsfClasses; c += 64u) {
          wave_sync();
          m.heads[c + lane_id()] = kNone;
        }
      }
      const uint32_t r0 = rec_take();
      push(r0, 0u, ag);
      ta.start(ag - 1u, r0);
    } else {
      frl = frh = 0u;
      ta.start(ag - 1u, ag);
    }
    if constexpr (kKeys) {
      tb.init(m.tb_l, m.tb_g, m.tb_n);
      tb.start(ag - 1u, ag);
    }
  }

  // First and next fit: the block at position p of chunk ci (row r current,
  // key e = its last granule, value s = its size) gives sg granules from its
  // low end.
  template <bool CHK>
  __device__ __forceinline__ int64_t commit_fit(uint32_t ci, uint32_t p, const Row& r,
                                                uint32_t e, uint32_t s, uint32_t sg) {
    const uint32_t a = e - s + 1u;
    live_push<CHK>(a, sg);
    if (likely(s > sg)) {
      ta.store_field(ta.slot(ci), p, 1u, s - sg);  // the end stays
      if (kMax) ta.shrink(ci, s, TA::with(r, p, e, s - sg));
    } else {
      ta.erase_at(ci, p, r);
      --F;
    }
    if (ALGO == kNextFit) rover = a + sg;
    return (int64_t)(uint64_t)a;
  }

  // Allocate sg granules; kreq is the request's byte class (segregated fit)
  // or request class (TLSF).  Returns the first granule, -1 or kENoMeta.
  __device__ __forceinline__ bool full_dir() const {
    return D < kOrdDir && (ta.nc >= 64u * D || (kKeys && tb.nc >= 64u * D));
  }

  // Where a heap that comes from the lean core leaves its free entries
  // (address, end) and their keys: the tops of the two table areas.
  __device__ __forceinline__ HDA_GLOBAL Ent* staged_ents(uint32_t f) const {
    return (HDA_GLOBAL Ent*)(m.tb_g - (uint64_t)f * 8u);
  }
  __device__ __forceinline__ HDA_GLOBAL uint32_t* staged_keys(uint32_t f) const {
    return (HDA_GLOBAL uint32_t*)(m.tb_g + (m.tb_g - m.ta_g) - (uint64_t)f * 4u);
  }
  // Write lean heap w's live entries and free entries (in table order) to
  // the device slot: its tables share the LDS this core is about to use.
  template <typename Lean>
  __device__ __forceinline__ void stage(const Lean& w) const {
    const uint32_t lane = lane_id();
    for (uint32_t base = 0; base < w.L; base += 64u) {
      const uint32_t i = base + lane;
      wave_sync();
      const Ent e = *w.live_ptr(i < w.L ? i : 0u);
      if (i < w.L) m.gl[i] = e;
    }
    HDA_GLOBAL Ent* const ents = staged_ents(w.F);
    HDA_GLOBAL uint32_t* const keys = staged_keys(w.F);
    w.each_chunk([&](uint32_t c, uint32_t a, uint32_t e, uint32_t k) {
      const uint32_t i = 64u * c + lane;
      if (i < w.F) {
        ents[i] = mk_ent(a, e);
        if (kSeg) keys[i] = k;
      }
    });
    wave_order();
  }
  // Start from f staged free entries and l staged live entries: each lane
  // finds the place of its entries in the sorted tables by counting the
  // entries below them (f^2 / 64 steps, about 0.1 ms at 500 free blocks,
  // once), and the chunks, records and first live entries go where this core
  // keeps them.  At most ord_adopt_max(capF) free blocks; chunk i is slot i.
  // kshift: the position of the class in a key.
  __device__ __forceinline__ void adopt(uint32_t f, uint32_t l0, uint32_t rov, uint32_t kshift) {
    const uint32_t lane = lane_id();
    F = f; L = l0; rover = rov;
    HDA_GLOBAL Ent* const ents = staged_ents(F);
    HDA_GLOBAL uint32_t* const keys = staged_keys(F);
    ta.init(m.ta_l, m.ta_g, m.ta_n);
    if constexpr (kKeys) tb.init(m.tb_l, m.tb_g, m.tb_n);
    // chunk i takes entries [i F / n, (i + 1) F / n): 32 to 64 of them each
    // when there are two or more
    const uint32_t n = F <= 64u ? 1u : (F + 55u) / 56u;
    for (uint32_t base = 0; base < F; base += 64u) {
      const uint32_t i = base + lane;
      const bool v = i < F;
      const uint32_t iv = v ? i : 0u;
      wave_sync();
      const Ent me = ents[iv];
      const uint32_t a = ent_a(me), e = ent_s(me), s = e - a, k = kSeg ? keys[iv] : 0u;
      // entries below this one by end; by (size, end) or by key
      uint32_t ra = 0, rb = 0;
      bool newer = false, older = false;  // in the same class list
      for (uint32_t d = 0; d < F; d += 64u) {
        const uint32_t t = d + lane < F ? d + lane : 0u;
        wave_sync();
        const Ent o = ents[t];
        const uint32_t ko = kSeg ? keys[t] : 0u;
        const uint32_t m1 = F - d < 64u ? F - d : 64u;
        for (uint32_t l = 0; l < m1; ++l) {
          const uint32_t ej = rdlane(ent_s(o), l);
          ra += ej < e ? 1u : 0u;
          if constexpr (kKeys) {
            const uint32_t sj = ej - rdlane(ent_a(o), l);
            rb += (sj < s || (sj == s && ej < e)) ? 1u : 0u;
          }
          if constexpr (kSeg) {
            const uint32_t kj = rdlane(ko, l);
            const bool list = (kj >> kshift) == (k >> kshift);
            rb += kj < k ? 1u : 0u;
            newer = newer || (list && kj < k);
            older = older || (list && kj > k);
          }
        }
      }
      if (v) {
        // a record's number is its rank by key: a class's blocks are
        // numbered one after another from the head
        place(m.ta_g, ra, n, e - 1u, kSeg ? rb : s);
        if constexpr (kKeys) place(m.tb_g, rb, n, e - 1u, s);
        if constexpr (kSeg) {
          u32x4 r;
          r[0] = a; r[1] = s;
          r[2] = older ? rb + 1u : kNone;
          r[3] = newer ? rb - 1u : kNone;
          m.rec_g[rb] = r;
        }
      }
    }
    wave_order();
    build(ta, n);
    if constexpr (kKeys) build(tb, n);
    hd = kNone; bm = 0ull; slb = 0u; frl = frh = 0u; spare = kNone;
    if constexpr (kSeg) {
      // free record numbers: F .. capF - 1
      const uint32_t b0 = 64u * lane;
      const uint64_t fr = lanes_below(capF > b0 ? capF - b0 : 0u) &
                          ~lanes_below(F > b0 ? F - b0 : 0u);
      frl = (uint32_t)fr;
      frh = (uint32_t)(fr >> 32);
      if constexpr (ALGO == kTlsf) {
        for (uint32_t c = 0; c < kTlsfClasses; c += 64u) {
          wave_sync();
          m.heads[c + lane] = kNone;
        }
      }
      for (uint32_t base = 0; base < F; base += 64u) {
        const uint32_t i = base + lane;
        const bool v = i < F;
        wave_sync();
        const u32x4 r = m.rec_g[v ? i : 0u];
        if (v && i < m.rec_n) m.rec_l[i] = r;
        const uint32_t c = cls(r[1]);
        uint64_t h = ballot(v && r[3] == kNone);
        for (; h != 0ull; h &= h - 1ull) {
          const uint32_t l = ctz64(h), cl = rdlane(c, l);
          set_head(cl, base + l);
          bit_set(cl);
        }
      }
    }
    for (uint32_t base = 0; base < L && base < m.ll_n; base += 64u) {
      const uint32_t i = base + lane;
      wave_sync();
      if (i < L && i < m.ll_n) m.ll[i] = m.gl[i];
    }
    wave_order();
  }
  // Entry (key, value) of rank r among F in n chunks, into chunk slot memory.
  __device__ __forceinline__ void place(HDA_GLOBAL uint8_t* g, uint32_t r, uint32_t n,
                                        uint32_t key, uint32_t val) const {
    const uint32_t c = ((r + 1u) * n - 1u) / F, p = r - c * F / n;
    u32x2 v;
    v[0] = key; v[1] = val;
    *(HDA_GLOBAL u32x2*)(g + (uint64_t)c * TA::CB + p * 8u) = v;
  }
  // Chunks 0 .. n - 1 from the slots place() filled, and their directory.
  template <typename T>
  __device__ __forceinline__ void build(T& t, uint32_t n) {
    for (uint32_t c = 0; c < n; ++c) {
      const uint32_t cnt = (c + 1u) * F / n - c * F / n;
      const bool in = lane_id() < cnt;
      wave_sync();
      const u32x2 v = *(const HDA_GLOBAL u32x2*)(t.gb + (uint64_t)c * T::CB + lane_id() * 8u);
      const typename T::Row r{in ? v[0] : kNone, in ? v[1] : T::kSentS};
      t.store(c, r);
      dir_put(t.dsl, c, c);
      t.describe(c, r, cnt);
    }
    t.nc = n;
#pragma unroll
    for (int k = 0; k < T::ND; ++k) t.used[k] = lanes_below(n > 64u * k ? n - 64u * k : 0u);
  }

  // Continue a heap that ran with fewer directory registers: the same
  // chunks, records and live entries, the directories widened.
  template <int D1>
  __device__ __forceinline__ void take(const OrdHeap<ALGO, D1>& o) {
    widen(ta, o.ta);
    if constexpr (kKeys) widen(tb, o.tb);
    F = o.F; L = o.L; rover = o.rover;
    hd = o.hd; bm = o.bm; slb = o.slb; frl = o.frl; frh = o.frh; spare = o.spare;
  }
  template <typename T2, typename T1>
  __device__ __forceinline__ static void widen(T2& t, const T1& o) {
    t.init(o.lb, o.gb, o.nl_req);
#pragma unroll
    for (int k = 0; k < T1::ND; ++k) {
      t.dsl[k] = o.dsl[k]; t.dct[k] = o.dct[k]; t.dk0[k] = o.dk0[k]; t.dk1[k] = o.dk1[k];
      t.dmx[k] = o.dmx[k]; t.used[k] = o.used[k];
    }
    t.nc = o.nc;
  }

  // CHK = false: block_safe holds for the current block, so no request of
  // it finds a table at the directory's limit or reaches a capacity.
  template <bool CHK = true>
  __device__ __forceinline__ int64_t alloc(uint32_t sg, uint32_t kreq) {
    if (CHK && full_dir()) return kOverflow;
    if constexpr (ALGO == kFirstFit) {
      const uint32_t ci = ta.first_fit_chunk(sg, 0u);
      if (ci == kNone) return fail<CHK>();
      const Row r = ta.load(ta.slot(ci));
      const uint32_t p = ctz64(ballot(r.s >= sg));
      const uint32_t e = rdlane(r.a, p), s = rdlane(r.s, p);
      if (CHK && L >= capL) return kENoMeta;
      return commit_fit<CHK>(ci, p, r, e, s, sg);
    } else if constexpr (ALGO == kNextFit) {
      // the search starts at the first block ending past the rover (R9-R11)
      // and runs on cyclically: the rest of that chunk, the later chunks,
      // then from the first chunk
      uint32_t ci, q0;
      Row r;
      ta.locate(0u, rover, ci, r, q0);
      uint32_t p;
      const uint64_t fit = ballot(r.s >= sg) & ~lanes_below(q0);
      if (likely(fit != 0ull)) {
        p = ctz64(fit);
      } else {
        const uint32_t c1 = ta.first_fit_chunk(sg, ci + 1u);
        const uint32_t c2 = c1 != kNone ? c1 : ta.first_fit_chunk(sg, 0u);
        if (c2 == kNone) return fail<CHK>();
        if (c2 != ci) r = ta.load(ta.slot(c2));
        ci = c2;
        p = ctz64(ballot(r.s >= sg));
      }
      const uint32_t e = rdlane(r.a, p), s = rdlane(r.s, p);
      if (CHK && L >= capL) return kENoMeta;
      return commit_fit<CHK>(ci, p, r, e, s, sg);
    } else if constexpr (ALGO == kBestFit) {
      // smallest key (size, last granule) at or above (sg, 0)
      uint32_t ci, p;
      typename TB::Row r;
      tb.locate(sg, 0u, ci, r, p);
      if (unlikely(p >= tb.count(ci))) {
        if (ci + 1u >= tb.nc) return fail<CHK>();
        ci = ci + 1u;
        r = tb.load(tb.slot(ci));
        p = 0u;
      }
      const uint32_t s = rdlane(r.s, p), e = rdlane(r.a, p);
      if (CHK && L >= capL) return kENoMeta;
      // the block's entry in the address table is looked up first: the key
      // table's updates do not touch it, and its load then overlaps them
      uint32_t cj, q;
      Row ra;
      ta.locate(0u, e + 1u, cj, ra, q);
      tb.erase_at(ci, p, r);
      if (likely(s > sg)) tb.insert_key(e, s - sg);
      return commit_fit<CHK>(cj, q - 1u, ra, e, s, sg);
    } else {
      // class of the first non-empty list at or above the request's
      uint32_t c;
      if constexpr (ALGO == kTlsf) {
        const uint32_t fl = kreq >> 5, sl = kreq & 31u;
        const uint32_t m2 = rdlane(slb, fl) & (~0u << sl);
        if (m2 != 0u) {
          c = (fl << 5) | (uint32_t)__builtin_ctz(m2);
        } else {
          const uint64_t m1 = fl < 63u ? bm & (~0ull << (fl + 1u)) : 0ull;
          if (m1 == 0ull) return fail<CHK>();
          const uint32_t f2 = ctz64(m1);
          c = (f2 << 5) | (uint32_t)__builtin_ctz(rdlane(slb, f2));
        }
      } else {
        // (a request no larger than the arena has a class below 64)
        const uint64_t mk = bm & (~0ull << kreq);
        if (mk == 0ull) return fail<CHK>();
        c = ctz64(mk);
      }
      const uint32_t i = head(c);
      const Rec b = rec(i);
      if (CHK && L >= capL) return kENoMeta;
      live_push<CHK>(b.a, sg);
      // pop the head (Alg. 4), keeping the lists' invariants (R20)
      set_head(c, b.nx);
      if (b.nx == kNone) bit_clear(c); else rec_link(b.nx, 3u, kNone);
      if (b.s > sg) {
        // the remainder, same record and same end, is pushed at the head of
        // its class (Alg. 4)
        push(i, b.a + sg, b.s - sg);
      } else {
        uint32_t ci, q;
        Row r;
        ta.locate(0u, b.a + b.s, ci, r, q);
        ta.erase_at(ci, q - 1u, r);
        rec_give(i);
        --F;
      }
      return (int64_t)(uint64_t)b.a;
    }
  }

  // Release [x, x + sz) into the free blocks, merging with free neighbours
  // (Alg. 2 / Alg. 5).  Returns false, changing nothing, when a new free
  // entry would exceed the capacity.
  template <bool CHK = true>
  __device__ __forceinline__ bool release(uint32_t x, uint32_t sz) {
    const uint32_t xe = x + sz;
    // the block whose last granule is x - 1 (an exact key) and the block
    // after x (the next entry, starting at xe if it borders)
    uint32_t ci, q;
    Row r;
    ta.locate(0u, x, ci, r, q);
    // best fit: where the freed part's own key goes if nothing merges, its
    // load beside the address table's
    uint32_t ck = 0, k = 0;
    typename TB::Row rk{0u, 0u};
    if constexpr (kKeys) tb.locate(sz, xe - 1u, ck, rk, k);
    const uint32_t p = q - 1u;
    const bool hasL = q != 0u && rdlane(r.a, p) + 1u == x;
    const uint32_t vl = rdlane(r.s, p);  // size or record (hasL)
    // the entry at position q, or the first one of the next chunk
    uint32_t rci = ci, rp = q;
    Row rr = r;
    bool next = true;
    if (unlikely(q >= ta.count(ci))) {
      next = ci + 1u < ta.nc;
      if (next) {
        rci = ci + 1u; rp = 0u;
        rr = ta.load(ta.slot(rci));
      }
    }
    const uint32_t er = rdlane(rr.a, rp), vr = rdlane(rr.s, rp);
    uint32_t sl = 0, sr = 0;
    Rec bl{0, 0, kNone, kNone}, br{0, 0, kNone, kNone};
    bool hasR;
    if constexpr (kSeg) {
      // the right record says whether its block borders
      const u32x4 qr = rec_raw(next ? vr : 0u);
      if (hasL) bl = rec(vl);
      br = rec_of(qr);
      sl = bl.s;
      sr = br.s;
      hasR = next && br.a == xe;
    } else {
      sl = vl;
      sr = vr;
      hasR = next && er + 1u - vr == xe;
    }
    if (CHK && !hasL && !hasR && F >= capF) return false;
    const uint32_t ma = hasL ? x - sl : x;
    const uint32_t ms = (hasL ? sl : 0u) + sz + (hasR ? sr : 0u);
    const uint32_t me = hasR ? er : xe - 1u;  // last granule of the merged block
    if constexpr (kSeg) {
      // unlink the free neighbours, then push the merged block (R21)
      if (hasL) {
        unlink(sl, bl.nx, bl.pv);
        // unlinking the left block rewrote the links of its list
        // neighbours, which may include the right block
        br.pv = br.pv == vl ? bl.pv : br.pv;
        br.nx = br.nx == vl ? bl.nx : br.nx;
      }
      if (hasR) unlink(sr, br.nx, br.pv);
    }
    if constexpr (kKeys) {
      if (hasL) tb.erase_key(x - 1u, sl);
      if (hasR) tb.erase_key(er, sr);
      if (hasL || hasR) tb.insert_key(me, ms);
      else tb.insert_at(ck, k, rk, typename TB::Row{me, ms});
    }
    if (hasL && hasR) {
      // the right block's entry keeps its end and takes the merged block;
      // the left block's entry goes
      if constexpr (kSeg) {
        push(vr, ma, ms);
        rec_give(vl);
      } else {
        ta.store_field(ta.slot(rci), rp, 1u, ms);
        if (rci == ci) r = TA::with(r, rp, er, ms);  // the row erase_at shifts
        if (kMax) ta.grow(rci, ms);
      }
      ta.erase_at(ci, p, r);
      --F;
    } else if (hasL) {
      // the left block's entry ends later now (its place does not change)
      const uint32_t v = kSeg ? vl : ms;
      ta.store_entry(ta.slot(ci), p, me, v);
      if (p == 0u) dir_put(ta.dk0, ci, me);
      if (kMax) ta.grow(ci, ms);
      if constexpr (kSeg) push(vl, ma, ms);
    } else if (hasR) {
      // the right block grows downwards: its end and its entry stay
      if constexpr (kSeg) {
        push(vr, ma, ms);
      } else {
        ta.store_field(ta.slot(rci), rp, 1u, ms);
        if (kMax) ta.grow(rci, ms);
      }
    } else {
      // a new entry at position q
      uint32_t v = sz;
      if constexpr (kSeg) {
        v = rec_take();
        push(v, x, sz);
      }
      ta.insert_at(ci, q, r, Row{me, v});
      ++F;
    }
    return true;
  }

  // Free live entry idx except its first floor(cut * size / 2^31) granules
  // (partial deallocation, sequential fits; cut < 2^31).  Returns the first
  // granule of the released part or kENoMeta.
  // v0, w0: the victim and the last live entry, as loaded.
  template <bool CHK = true>
  __device__ __forceinline__ int64_t free_index(uint32_t idx, Ent v0, Ent w0, uint32_t cut) {
    const Ent v = mk_ent(uniform(ent_a(v0)), uniform(ent_s(v0)));
    const uint32_t bx = ent_a(v), bsz = ent_s(v);
    const uint32_t t = (kSeg || cut == 0u) ? 0u : (uint32_t)(((uint64_t)cut * bsz) >> 31);
    const uint32_t x = bx + t, sz = bsz - t;
    // the live table does not depend on the free one: without checks it is
    // brought up to date first, and the next request's victim is on its way
    // while this one's part is released
    if (CHK && !release<CHK>(x, sz)) return kENoMeta;
    if (t != 0u) {
      lset(idx, mk_ent(bx, t));
    } else {
      lset(idx, w0);
      --L;
    }
    if (!CHK) {
      look_ahead();
      release<CHK>(x, sz);
    }
    return (int64_t)(uint64_t)x;
  }

  template <bool CHK = true>
  __device__ __forceinline__ int64_t free_draw(uint32_t r, uint32_t cut) {
    if (CHK && L == 0u) return kFail;
    if (CHK && full_dir()) return kOverflow;
    const uint32_t idx = (uint32_t)(((uint64_t)r * (uint64_t)L) >> 32);
    if constexpr (CHK) {
      const Ent v0 = lraw(idx), w0 = lraw(L - 1u);  // both loaded before either is used
      return free_index<CHK>(idx, v0, w0, cut);
    } else {
      return free_index<CHK>(idx, nv, nw, cut);
    }
  }

  // The victim of the next request, if that is a free, and the last live
  // entry are loaded as soon as the live table is as that request will find
  // it (blocks without checks): their latency, which nothing else hides from
  // a lone wave, then overlaps the rest of the current request.
  uint32_t nr;       // the next request's draw
  bool nfree;        // it is a free
  Ent nv, nw;        // its victim, the last live entry
  __device__ __forceinline__ void next_request(bool is_free, uint32_t draw) {
    nfree = is_free;
    nr = draw;
  }
  __device__ __forceinline__ void look_ahead() {
    if (nfree) {
      nv = lraw((uint32_t)(((uint64_t)nr * (uint64_t)L) >> 32));
      nw = lraw(L != 0u ? L - 1u : 0u);
    }
  }
  template <bool CHK>
  __device__ __forceinline__ int64_t fail() {  // nothing fits
    if (!CHK) look_ahead();
    return kFail;
  }
  template <bool CHK>
  __device__ __forceinline__ void live_push(uint32_t a, uint32_t sg) {
    lset(L, mk_ent(a, sg));
    ++L;
    if (!CHK) look_ahead();
  }

  // Whether the next n requests can skip the directory and capacity checks:
  // each adds at most one live entry and one free block, so none of them
  // reaches a capacity, and with n live blocks to start from no free finds
  // the live table empty.  Every chunk of a table holds at least 32 entries
  // once there are two, so a table with fewer than 32 x 64 D free blocks has
  // fewer than 64 D chunks: with F + n below that, no request starts with a
  // table at the directory's limit.  (With the widest directory there is no
  // directory check.)
  __device__ __forceinline__ bool block_safe(uint32_t n) const {
    return L + n <= capL && F + n <= capF && L >= n &&
           (D >= kOrdDir || F + n < 32u * 64u * D);
  }
  __device__ __forceinline__ void set_room() {}  // nothing to refresh after a block

  // Canonical state (format in hda.h).
  __device__ __forceinline__ int64_t dump(int64_t* out, int64_t cap) {
    const uint32_t lane = lane_id();
    const int64_t lists = ALGO == kTlsf ? kTlsfClasses : (ALGO == kSegFit ? 64 : 0);
    const int64_t need = 4 + 2 * (int64_t)F + 2 * (int64_t)L + (kSeg ? lists + (int64_t)F : 0);
    if (out == nullptr || need > cap) return need;
    const uint32_t sh = shift;
    wave_sync();
    if (lane == 0) out[0] = F;
    int64_t* fo = out + 1;
    uint32_t k = 0;
    for (uint32_t ci = 0; ci < ta.nc; ++ci) {
      const Row r = ta.load(ta.slot(ci));
      const uint32_t n = ta.count(ci);
      uint32_t a = r.a + 1u - r.s, s = r.s;
      if constexpr (kSeg) {
        // this lane's record (lanes past the chunk read record 0, unused)
        wave_sync();
        const uint32_t i = lane < n && r.s < kOrdMaxFree ? r.s : 0u;
        u32x4 v;
        if (i < m.rec_n) v = m.rec_l[i]; else v = m.rec_g[i];
        a = v[0];
        s = v[1];
      }
      wave_sync();
      if (lane < n) {
        fo[2 * (k + lane)] = (int64_t)((uint64_t)a << sh);
        fo[2 * (k + lane) + 1] = (int64_t)((uint64_t)s << sh);
      }
      k += n;
    }
    int64_t* lo = out + 1 + 2 * (int64_t)F;
    wave_sync();
    if (lane == 0) lo[0] = L;
    for (uint32_t base = 0; base < L; base += 64u) {
      const Ent e = lchunk(base);
      const uint32_t i = base + lane;
      wave_sync();
      if (i < L) {
        lo[1 + 2 * i] = (int64_t)((uint64_t)ent_a(e) << sh);
        lo[2 + 2 * i] = (int64_t)((uint64_t)ent_s(e) << sh);
      }
    }
    int64_t* tail = lo + 1 + 2 * (int64_t)L;
    wave_sync();
    if (lane == 0) {
      tail[0] = ALGO == kNextFit ? (int64_t)((uint64_t)rover << sh) : -1;
      tail[1] = kSeg ? (int64_t)bm : 0;
    }
    if constexpr (kSeg) {
      // each class: its length, then its blocks from the head along the
      // next links (bounded by the section's words even if a list were
      // corrupt)
      int64_t* ls = tail + 2;
      uint32_t pos = 0;
      for (uint32_t c = 0; c < (uint32_t)lists; ++c) {
        bool nonempty;
        if constexpr (ALGO == kTlsf) nonempty = (rdlane(slb, c >> 5) >> (c & 31u)) & 1u;
        else nonempty = (bm >> c) & 1ull;
        uint32_t n = 0;
        if (nonempty) {
          uint32_t i = head(c);
          while (i != kNone && pos + 1u + n < (uint32_t)lists + F) {
            const Rec b = rec(i);
            wave_sync();
            if (lane == 0) ls[pos + 1u + n] = (int64_t)((uint64_t)b.a << sh);
            i = b.nx;
            ++n;
          }
        }
        wave_sync();
        if (lane == 0) ls[pos] = n;
        pos += 1u + n;
      }
    }
    return need;
  }
};

}  // namespace hda
