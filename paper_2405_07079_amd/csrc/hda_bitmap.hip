// Batched replay of bitmask-allocator heaps (Sec. III-B), one wavefront per
// heap, waves pulling heaps from a queue in the caller's order.
//
// A heap is replayed from the table of its free runs (the lean core,
// hda_lean.h) in the wave's share of LDS, and moves to its granule flags and
// node summaries (hda_bitmap.h) in the wave's workspace slot when the tables
// outgrow that share.  Both give the same answers.  The flags are bound by
// the vector instructions that keep the summaries (120 per request); the
// table's answer is one test of the block at the rover, or one scan of a few
// 64-entry chunks: 4,096 heaps of 16 MiB at 64 B, 40,000 requests each, in
// 19.9 ms against 51.0 ms on the flags.  Heaps that move after a quarter of
// their trace (1,024 heaps, 20,000 requests, blocks to 4 or 16 KiB) still gain
// 1.13x from the part before, and 4,096 of them 1.14x.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "hda.h"
#include "hda_wave.h"
#include "hda_core.h"
#include "hda_replay_body.h"

using namespace hda;

namespace {

constexpr uint32_t kWavesPerGroup = 4;
constexpr int64_t kMaxWaves = 4096;
// LDS per wave, which keeps four waves per SIMD: the pool of the heap's free
// and live tables; a heap that outgrows it continues on its flags, with the
// summaries of the first kLdsNodes nodes (a 16 MiB heap of 64 B granules has
// 64) and the first live entries in the same bytes
constexpr uint32_t kLdsNodes = 64;
constexpr uint32_t kLdsWaveBytes = 10240;
// the workspace starts with the heap queue's counter and the moved heaps'
// (256 bytes)
constexpr uint64_t kHeaderBytes = 256;

// Workspace words of one wave's slot: the flags of max_granules, their node
// summaries (one per 64 words), then the live table.
__host__ __device__ uint64_t flag_words(uint64_t max_granules) { return (max_granules + 63u) / 64u; }
__host__ __device__ uint64_t node_words(uint64_t max_granules) { return (flag_words(max_granules) + 63u) / 64u; }
uint64_t slot_words(uint64_t max_granules, int64_t cap_live) {
  return flag_words(max_granules) + node_words(max_granules) + (uint64_t)cap_live;
}

int64_t n_waves(int64_t heaps) { return heaps < kMaxWaves ? heaps : kMaxWaves; }

// The queue counter and, after it, the count of heaps that moved to the flags
// start at 0 (a kernel rather than a memset, so the pair of launches can be
// captured in a graph).
__global__ void bitmap_reset(uint32_t* queue) {
  if (threadIdx.x < 2) queue[threadIdx.x] = 0u;
}

struct BitmapParams {
  ReplayParams p;
  uint64_t* ws;
  uint64_t max_granules;
  uint64_t words;  // of a wave's slot
  int64_t waves;
};
typedef const __attribute__((address_space(4))) BitmapParams* LaunchParams;

// The two parts of a heap's replay as functions of their own, each compiled by
// itself: in one function the flags part, which most heaps never reach, took
// registers from the table's request loop (2 % on 4,096 heaps).  At most two
// calls a heap.  Arguments are wave-uniform but for BitmapExit's chunks; the
// kernel's parameters are read from where the launch put them.
struct WaveEnv {
  BitmapParams b;
  LeanLds lds;
  __device__ __forceinline__ WaveEnv(LaunchParams lp, uint32_t pool) {
    __builtin_memcpy(&b, (const void*)(LaunchParams)uniform64((uint64_t)lp), sizeof(b));
    lds.base = (HDA_LDS uint8_t*)(uintptr_t)uniform(pool);
    lds.bytes = kLdsWaveBytes;
  }
};
__device__ __attribute__((noinline)) BitmapExit table_call(LaunchParams lp, uint32_t pool,
                                                           uint32_t heap) {
  const WaveEnv e(lp, pool);
  return bitmap_start(e.b.p, e.lds, e.b.max_granules, (int64_t)uniform(heap));
}
__device__ __attribute__((noinline)) void flags_call(LaunchParams lp, uint32_t pool,
                                                     uint32_t wave, uint32_t heap, BitmapExit x) {
  const WaveEnv e(lp, pool);
  uint64_t* bits = e.b.ws + kHeaderBytes / 8u + (uint64_t)uniform(wave) * e.b.words;
  uint64_t* nodes = bits + flag_words(e.b.max_granules);
  Ent* live = reinterpret_cast<Ent*>(nodes + node_words(e.b.max_granules));
  x.st = (int32_t)uniform((uint32_t)x.st);
  x.pos = (int64_t)uniform64((uint64_t)x.pos);
  x.F = uniform(x.F); x.L = uniform(x.L); x.rover = uniform(x.rover);
  bitmap_continue(e.b.p, e.lds, bits, nodes, live, kLdsNodes, (int64_t)uniform(heap), x);
}

__global__ __launch_bounds__(64 * kWavesPerGroup) void bitmap_kernel(BitmapParams b) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const uint32_t wl = uniform(threadIdx.x / 64u);
  const uint32_t wave = uniform(blockIdx.x * kWavesPerGroup + wl);
  if ((int64_t)wave >= b.waves) return;
  const uint32_t pool = (uint32_t)(uintptr_t)((HDA_LDS uint8_t*)smem) + wl * kLdsWaveBytes;
  const LaunchParams lp = (LaunchParams)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t* queue = reinterpret_cast<uint32_t*>(b.ws);
  // a wave takes at most every heap, so the loop ends even if the queue were
  // never to run dry; every lane runs the atomic (lane 0 adds 1) so the value
  // read back does not come from a lane-dependent branch
  for (int64_t taken = 0; taken < b.p.n_heaps; ++taken) {
    uint32_t i = atomicAdd(queue, lane_id() == 0 ? 1u : 0u);
    i = rdlane(i, 0);
    if ((int64_t)i >= b.p.n_heaps) break;
    const uint32_t heap = b.p.order ? (uint32_t)b.p.order[i] : i;
    const BitmapExit x = table_call(lp, pool, heap);
    if (uniform((uint32_t)x.next)) flags_call(lp, pool, wave, heap, x);
  }
}

bool desc_ok(const hda_batch_desc* d, uint64_t max_granules) {
  if (!d || d->n_heaps < 0 || max_granules == 0 || max_granules >= (uint64_t(1) << 32) ||
      d->meta_live <= 0 || d->meta_live > (int64_t(1) << 31))
    return false;
  if (d->n_heaps == 0) return true;
  if (!d->arena || !d->align || !d->algo || !d->req_off || !d->req || !d->res || !d->status)
    return false;
  if (d->state && (!d->state_off || !d->state_len)) return false;
  return true;
}

}  // namespace

extern "C" {

size_t hda_bitmap_workspace(const hda_batch_desc* d, uint64_t max_granules) {
  if (!desc_ok(d, max_granules)) return 0;
  return (size_t)(n_waves(d->n_heaps) * slot_words(max_granules, d->meta_live) * 8u) +
         kHeaderBytes + 256u;
}

int hda_bitmap_replay(const hda_batch_desc* d, uint64_t max_granules, void* stream) {
  if (!desc_ok(d, max_granules)) return HDA_E_INVAL;
  if (d->n_heaps == 0) return HDA_OK;
  const size_t need = hda_bitmap_workspace(d, max_granules);
  if (!d->workspace || d->workspace_bytes < need) return HDA_E_RANGE;
  BitmapParams b;
  std::memset(&b, 0, sizeof(b));
  ReplayParams& p = b.p;
  p.arena = d->arena; p.align = d->align; p.algo = d->algo;
  p.req_off = d->req_off; p.req = d->req; p.res = d->res; p.order = d->order;
  p.state = d->state; p.state_off = d->state_off; p.state_len = d->state_len;
  p.status = d->status;
  p.n_heaps = d->n_heaps;
  p.cap_live = (uint32_t)d->meta_live;
  uintptr_t base = reinterpret_cast<uintptr_t>(d->workspace);
  base = (base + 255u) & ~uintptr_t(255);
  b.ws = reinterpret_cast<uint64_t*>(base);
  p.migrated = reinterpret_cast<uint32_t*>(base) + 1;
  b.max_granules = max_granules;
  b.words = slot_words(max_granules, d->meta_live);
  b.waves = n_waves(d->n_heaps);
  const uint32_t groups = (uint32_t)((b.waves + kWavesPerGroup - 1) / kWavesPerGroup);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(bitmap_reset, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(base));
  if (hipGetLastError() != hipSuccess) return HDA_E_DEVICE;
  hipLaunchKernelGGL(bitmap_kernel, dim3(groups), dim3(64 * kWavesPerGroup),
                     kLdsWaveBytes * kWavesPerGroup, s, b);
  return hipGetLastError() == hipSuccess ? HDA_OK : HDA_E_DEVICE;
}

}  // extern "C"
