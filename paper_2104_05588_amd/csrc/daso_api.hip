// C-ABI entry points of the DASO synchronisation library that touch the GPU:
// the per-stream statistics workspace, bucket grouping and launches.  Argument
// checking is in daso_host.cpp.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <utility>

#include "daso_host.h"
#include "daso_launch.h"

namespace {

// Kernel arguments are passed by value and limited to 4 KB.
static_assert(sizeof(daso::StepArgs) <= 4096, "StepArgs must fit the 4 KB kernel-argument limit");

using daso::StepArgs;
using daso::BucketSlots;
using daso::Group;
using daso::Ranges;
using daso::SlicePartial;

// ---------------------------------------------------------------- workspace
// Per (device, stream): the counter of launches that sum their own statistics
// (kStatsCounterBytes), the table of a fused call's buckets and the statistics
// partials of its workgroups.  Allocated on first use and
// replaced by one at least twice as large when a larger launch needs it.  A
// replaced buffer is never freed: launches already queued, and graphs captured
// earlier, may still use it; the doubling keeps the total within twice the
// largest buffer.  The counter is zeroed once, by a kernel that the first
// eager (not captured) call needing it queues on the stream, and every launch
// that uses it leaves it at zero; every launch writes each partial and table
// entry it later reads, so the rest never needs clearing.  A call holds the
// entry's lock
// from choosing the buffer until its last launch is queued, so that two host
// threads sharing a stream cannot queue one call's step between the other
// call's step and its statistics pass.
struct Workspace {
  std::mutex mu;
  void* ptr = nullptr;
  size_t bytes = 0;
  bool counter_zeroed = false;  // the zeroing of ptr's counter is queued on the stream
};

std::mutex g_ws_mu;  // guards the map itself; nodes never move or go away
std::map<std::pair<int, hipStream_t>, Workspace> g_ws;

Workspace& workspace_entry(int dev, hipStream_t stream) {
  std::lock_guard<std::mutex> lock(g_ws_mu);
  return g_ws[{dev, stream}];
}

// With w.mu held: make w hold at least `need` bytes.
int reserve(Workspace& w, size_t need) {
  if (w.bytes < need) {
    const size_t bytes = std::max<size_t>({need, 2 * w.bytes, size_t(1) << 20});
    void* p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return DASO_EHIP;
    w.ptr = p;  // the previous buffer, if any, stays allocated (see above)
    w.bytes = bytes;
    w.counter_zeroed = false;
  }
  return DASO_OK;
}

// With w.mu held, from an eager call: queue the zeroing of w's counter on
// `stream` once per buffer, before any launch that uses it.
int zero_counter_once(Workspace& w, hipStream_t stream) {
  if (w.counter_zeroed) return DASO_OK;
  if (daso::clear_stats_counter(w.ptr, stream) != hipSuccess) return DASO_EHIP;
  w.counter_zeroed = true;
  return DASO_OK;
}

// ---------------------------------------------------------- fixed scratch
// The statistics scratch of daso_fused_sync_step_noalloc: one array of fixed
// size in device memory, of which every GPU the library runs on holds its own
// copy until the process ends.  In host code `scratch` names a host-side stand-in,
// not device memory: the device address is looked up once per device with
// hipGetSymbolAddress (with that device current) and only that address is
// handed to kernels.  It has the workspace's layout, but its first
// kStatsCounterBytes are never used: calls through it keep the statistics
// kernel (see launch_groups).  The kernels write every partial and table entry
// they read later, so the array never needs clearing.
// The limit that callers see counts the tiles of the tiled plan, of 2048 or 1024 parameters;
// the array holds the partials, one per 1024 or 2048 parameters, of one launch at a time
// or of all, and a bucket that needs more takes several launches.
constexpr size_t kScratchBytes = DASO_NOALLOC_SCRATCH_BYTES;
static_assert(sizeof(SlicePartial) == daso::kPartialBytes && sizeof(BucketSlots) == daso::kEntryBytes,
              "the sizes that the cut of a call counts with");
static_assert(kScratchBytes % 256 == 0, "the scratch size is a whole number of 256-byte blocks");
static __device__ __align__(256) uint64_t scratch[kScratchBytes / sizeof(uint64_t)];

constexpr int kMaxDevices = 64;

struct ScratchSlot {
  std::once_flag once;
  hipError_t err = hipSuccess;
  void* ptr = nullptr;
  std::mutex mu;  // held by a call from choosing the buffer until its last launch is queued
};
ScratchSlot g_scratch[kMaxDevices];

// The device address of `scratch` on device `dev`, which must be current.
int scratch_slot(int dev, ScratchSlot** out) {
  if (dev < 0 || dev >= kMaxDevices) return DASO_EHIP;
  ScratchSlot& s = g_scratch[dev];
  std::call_once(s.once, [&s] { s.err = hipGetSymbolAddress(&s.ptr, HIP_SYMBOL(scratch)); });
  if (s.err != hipSuccess || s.ptr == nullptr) return DASO_EHIP;
  *out = &s;
  return DASO_OK;
}

// -------------------------------------------------------------- launching
// The launch's buckets as kernel arguments.
void fill_group(StepArgs& a, const Ranges& r, const Group& g, int shift) {
  a.cont = g.lo > r[g.first].start ? 1 : 0;
  for (int32_t k = 0; k < g.count; ++k) {
    const daso::Range& x = r[g.first + k];
    const int32_t d = 2 * x.S + a.P;
    a.start[k] = k == 0 ? g.lo : x.start;
    a.S[k] = x.S;
    a.inv[k] = d > 0 ? 1.0f / static_cast<float>(d) : 0.0f;
    a.out[k] = x.out;
  }
  a.start[g.count] = g.hi;
  a.nb = g.count;
  a.lo = g.lo;
  a.hi = g.hi;
  a.sb0 = g.lo >> shift;
  a.nslices = 8 * daso::superblocks(g.lo, g.hi, shift);
}

// A non-negative integer from the environment, read once per variable by the
// caller's static; `fallback` when unset, malformed or above `max`.
int64_t env_count(const char* name, int64_t fallback, int64_t max) {
  const char* e = getenv(name);
  if (e == nullptr || *e == '\0') return fallback;
  char* end = nullptr;
  const long long x = strtoll(e, &end, 10);
  return (end != e && *end == '\0' && x >= 0 && x <= max) ? static_cast<int64_t>(x) : fallback;
}

// DASO_FUSED_WG_PER_CU, when set, replaces the workgroups per CU of fused
// launches (0: no cap) and of the tiled plan; DASO_FUSED_RUN_ELEMS, a number of
// elements, replaces the run length of the tiled plan (0: plain order).  Neither
// changes a result.  Each is read once per process.
int64_t fused_run_elems_override() {
  static const int64_t v = env_count("DASO_FUSED_RUN_ELEMS", -1, int64_t(1) << 30);
  return v;
}
int64_t fused_cap_override() {
  static const int64_t v = env_count("DASO_FUSED_WG_PER_CU", -1, 64);
  return v;
}

// The average bucket up to which a launch takes wavefronts of each bucket's own
// (daso::small_buckets) in place of pieces and superblocks: where they win at every size
// up to it.  us per call in pieces and in buckets, all of one size:
//  - with statistics, 1M elements, g = 4, P = 8: buckets of 701 elements 172 and 73, 1001 117 and 56;
//    g = 8, P = 32: 350 and 114, 234 and 90; g = 4, P = 64: 254 and 168, 181 and 133; but
//    4M in buckets of 1500, g = 4, P = 64: 364 and 545; of 3001, g = 4, P = 8: 109 and 166;
//  - with statistics and unbounded counts, g = 9, P = 40, 4M in buckets of 1501 1036 and 446,
//    3001 413 and 326, 4096 210 and 304; 8192 elements in two buckets 12.2 and 23.2;
//  - without, 262144 elements, g = 4, P = 8: 63 elements 251 and 176, 200 60 and 56;
//    g = 4, P = 64: 462 and 414, 100 229 and 243;
//  - without, unbounded counts, g = 9, P = 40, 4M in buckets of 1501 420 and 268, 2001 336 and
//    219, 4096 136 and 140.
int64_t small_average_of(bool with_stats, const daso::Shape& shape) {
  const bool unbounded = shape.counts == daso::Counts::kUnbounded;
  if (with_stats) return unbounded ? 3072 : 1024;
  return unbounded ? 2048 : 64;
}

// LDS per workgroup, which caps how many workgroups share a CU.  By the bytes B
// that an element is read with; the best caps on MI355X, 25.6M (and, but for the
// fused step, 70.5M) parameters:
//  - workgroups of one wavefront: 190 / B of them for the fused step, 240 / B for
//    averages and merges, 5 to 16.  g = 1, P = 0 (B = 12): 87 us at 16, 92 at 8; g = 4, P = 0
//    (24): 132 at 8, 135 at 12, 145 at 20; g = 4, P = 8 (40): 197 at 5, 200 at 10, 213 at 20;
//    g = 8, P = 8 (56): 266 at 5, 278 at 10.  Averages of 3, 4 and 8 gradients: best
//    at 16, 16 and 8; merges of 4, 8 and 16 copies at 16, 12 and 8.  Averages and merges of
//    up to 8 bytes are not capped: 16 such workgroups have too little in flight (averages
//    of 1 and 2 gradients 31.3 and 46.4 us, 36.1 and 48.0 at 16; merges of 1 and 2 copies
//    41.4 and 46.4, 47.9 and 53.1; the mean of 1 to 4 copies 29 to 47, 44 to 54).
//  - the same with bounded counts, whose loads wait for more branches: 300 / B, 6 to 16,
//    5 beyond B = 80 (g = 3, P = 5, B = 30: 157 us at 10, 164 at 8, 187 at 6; g = 8, P = 12,
//    64: 297 at 6, 305 at 5 and 8; g = 8 with 12 fp32 copies, 88: 416 at 5, 427 at 6).
//  - with unbounded counts, which have a batch of streams in flight: 10 where bf16
//    copies are the most (g = 3, P = 40: 459 us, 510 at 7, 485 at 16), else 7 (g = 16, P = 8:
//    400, 413 at 10, 438 at 16; g = 4 with 40 fp32 copies: 825, 853 and 905).
//  - workgroups of four, with statistics: 4 up to B = 12 (92 us; 95 with 3), 3 up to
//    36 (g = 4, P = 4: 177 us; 186 with 2, 180 with 4), else 2 (g = 8, P = 0: 204;
//    219 with 3); with bounded counts 4 up to 22 (g = P = 1: 106 us, 118 with 3; g = 2, P = 3:
//    133 and 136; g = 3, P = 2, B = 24: 141 and 139); unbounded counts as above 3 (478 us;
//    522 with 2, 501 with 4) or 2 (425; 444 with 3), and 1 beyond B = 128 (g = 8 with 32 fp32 copies: 745; 817 with
//    2; registers hold P = 64 there by themselves).
//  - workgroups of eight: 1.
//  - workgroups of four, without: 1 (g = 8, P = 32: 473 us against 499 with 2); for the merge
//    of 32 bf16 copies 3 (289; 298 with 2, 341 with 1), for their mean 2 (263; 270 with 3).
//  - the pack (B = 4) needs the whole chip (24 us; 32 us with 16 wavefronts per CU).
// A call of up to 3M elements is not capped: its launch is over before the front has
// spread, and a cap leaves it in more rounds than need be (g = 4, P = 8 without statistics,
// capped and not: 0.5M elements 6.1 and 5.5 us, 1M 11.5 and 10.5, 2M 18.3 and 17.6, 4M
// 34.3 and 34.0, 8M 63.9 and 66.4).  The launches of a longer call are capped whatever
// their own size.
// DASO_FUSED_WG_PER_CU replaces the count for the fused step (0: no cap).
int32_t lds_of(daso::Mode mode, bool with_stats, const daso::Shape& shape, const StepArgs& a, int64_t elems) {
  if (mode == daso::kModePack) return 0;
  const int64_t over = fused_cap_override();
  if (mode == daso::kModeFused && over >= 0) return daso::lds_for_workgroups_per_cu(static_cast<int32_t>(over));
  int32_t bytes = a.P * (a.xf32 ? 4 : 2);
  if (mode == daso::kModeAvg) bytes = 4 * a.g;
  if (mode == daso::kModeMerge) bytes += 4;
  if (mode == daso::kModeFused) bytes += 4 * a.g + 8;
  if (elems <= daso::kShortCall) return 0;
  const bool unbounded = shape.counts == daso::Counts::kUnbounded;
  const bool mostly_bf16 = !a.xf32 && a.P > a.g;
  const auto share = [bytes](int32_t of, int32_t least) { return std::min(16, std::max(least, (of + bytes / 2) / bytes)); };
  int32_t per_cu = 1;
  if (mode != daso::kModeFused && bytes <= 8) return 0;
  if (shape.waves == 1) {
    if (unbounded) per_cu = mostly_bf16 ? 10 : 7;
    else if (shape.counts == daso::Counts::kBounded) per_cu = share(300, bytes > 80 ? 5 : 6);
    else per_cu = share(mode == daso::kModeFused ? 190 : 240, 5);
  } else if (with_stats && shape.waves == 4) {
    if (unbounded) per_cu = mostly_bf16 ? 3 : 2;
    else per_cu = bytes <= (shape.counts == daso::Counts::kBounded ? 22 : 12) ? 4 : bytes <= 36 ? 3 : bytes <= 128 ? 2 : 1;
  } else if (mode != daso::kModeFused && !a.xf32) {
    per_cu = mode == daso::kModeMean ? 2 : 3;
  }
  return daso::lds_for_workgroups_per_cu(per_cu);
}

// The current device, which must also be the device of `stream` (kernels run
// on the stream's device and the buffers and workspace live on the current one).
int current_device(hipStream_t stream, int* dev) {
  if (hipGetDevice(dev) != hipSuccess) return DASO_EHIP;
  if (stream == nullptr) return DASO_OK;
  hipDevice_t sdev = 0;
  if (hipStreamGetDevice(stream, &sdev) != hipSuccess) return DASO_EHIP;
  return sdev == *dev ? DASO_OK : DASO_EINVAL;
}

// Where a fused launch with statistics keeps its partials and table.
enum class Space {
  kAllocated,  // the per-(device, stream) workspace, allocated on first use
  kFixed,      // the fixed `scratch` array; calls needing more fail with DASO_ENOSPACE
};

int launch_groups(daso::Mode mode, StepArgs& a, const daso_bucket* b, int32_t nb,
                  daso_bucket_stats* stats, hipStream_t stream, Space space) {
  const bool with_stats = (mode == daso::kModeFused) && stats != nullptr;
  const Ranges ranges(b, nb, with_stats);
  const int64_t n = ranges[ranges.size() - 1].end;
  // The limits that are stated in tiles: of the no-alloc entry point's scratch, and 2^31 of them
  // for 64 buckets, which fewer than 2^40 elements cannot reach.
  if ((with_stats && space == Space::kFixed) || n >= int64_t(1) << 40) {
    const int64_t tile = daso::plan_tile(mode, a.g, a.P, a.xf32 != 0);
    int64_t max_tiles = 1;
    for (int32_t i = 0; i < nb; i += daso::kPlanBuckets)
      max_tiles = std::max(max_tiles, daso::plan_tiles(b, nb, i, tile));
    if (max_tiles > INT32_MAX) return DASO_EINVAL;
    if (with_stats && space == Space::kFixed && daso::plan_scratch(max_tiles) > DASO_NOALLOC_SCRATCH_BYTES)
      return DASO_ENOSPACE;
  }
  int dev = 0;
  const int drc = current_device(stream, &dev);
  if (drc != DASO_OK) return drc;
  // the plain average, in the form that finishes a blocking synchronisation: the wire went
  // out before it, so a merge that packs one as well keeps the merge's instances
  if (mode == daso::kModeMerge && a.P > 0 && a.wire == nullptr && ranges.size() == 1 && ranges[0].S == 0)
    mode = daso::kModeMean;
  a.n = n;
  for (int32_t r = 0; a.gavg != nullptr && r < a.g; ++r) a.in_place_avg |= a.grads[r] == a.gavg ? 1 : 0;
  a.g_inv = a.g > 0 ? 1.0f / static_cast<float>(a.g) : 0.0f;
  const daso::Shape shape = daso::launch_shape(mode, with_stats, a);
  const int shift = daso::super_shift(shape.waves);
  const uint32_t lds = static_cast<uint32_t>(lds_of(mode, with_stats, shape, a, n));
  // statistics scratch: the counter, the bucket table, the partials
  const int64_t counter_bytes = static_cast<int64_t>(daso::kStatsCounterBytes);
  daso::Cut cut;
  if (!with_stats) cut = daso::cut_of(ranges, shift, false, 0);
  std::unique_lock<std::mutex> hold;
  uint32_t* counter = nullptr;
  if (with_stats) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusActive;
    const bool capturing = hipStreamIsCapturing(stream, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone;
    void* base = nullptr;
    if (space == Space::kFixed) {
      ScratchSlot* slot = nullptr;
      const int rc = scratch_slot(dev, &slot);
      if (rc != DASO_OK) return rc;
      hold = std::unique_lock<std::mutex>(slot->mu);
      base = slot->ptr;
      cut = daso::cut_of(ranges, shift, true, static_cast<int64_t>(kScratchBytes) - counter_bytes);
    } else {
      Workspace& w = workspace_entry(dev, stream);
      hold = std::unique_lock<std::mutex>(w.mu);
      // a captured call cannot allocate: it makes do with what an eager call over as many
      // elements left, if need be in a pass per launch, which gives the same bits
      const int64_t least = daso::least_bytes(n), held = static_cast<int64_t>(w.bytes) - counter_bytes;
      cut = daso::cut_of(ranges, shift, true, capturing && held >= least ? held : least + daso::kSharedBytes);
      const int64_t shared = cut.pass_each ? 0 : cut.table * daso::kEntryBytes + cut.slots * daso::kPartialBytes;
      const int rc = reserve(w, static_cast<size_t>(counter_bytes + std::max(least, shared)));
      if (rc != DASO_OK) return rc;
      base = w.ptr;
      // the last-workgroup statistics of small eager launches count in w's counter
      if (!capturing) {
        const int zc = zero_counter_once(w, stream);
        if (zc != DASO_OK) return zc;
        counter = static_cast<uint32_t*>(base);
      }
    }
    a.table = reinterpret_cast<BucketSlots*>(static_cast<char*>(base) + counter_bytes);
    a.partials = reinterpret_cast<SlicePartial*>(a.table + cut.table);
    a.stats = stats;
  }
  BucketSlots* const table = a.table;
  const int64_t small_average = small_average_of(with_stats, shape);
  int64_t from = -1;
  bool partials = false;  // some launch so far leaves its statistics to a pass
  for (int32_t i = 0; i < ranges.size();) {
    const Group g = daso::cut_to(daso::group_at(ranges, i, shift, cut.room, from), shift, cut.room);
    const bool whole = g.hi == ranges[i + g.count - 1].end;
    fill_group(a, ranges, g, shift);
    // an eager call of few workgroups sums its own statistics in its last one,
    // which saves a launch's host cost (about 2.6 us); a graph replays launches without
    // that host cost, so a captured call keeps the statistics kernel (counter
    // stays null), and so does the no-alloc entry point, whose scratch every
    // call on the GPU shares: two of its calls racing on another stream could
    // leave a counter wrong for later calls, not only their own statistics
    a.done = cut.launches == 1 && a.nslices * shape.waves <= daso::kFinishStatsMaxWaves ? counter : nullptr;
    const int64_t row = daso::host::launch_grid(a.nslices, 1);
    const dim3 grid(static_cast<uint32_t>(row), static_cast<uint32_t>((std::max<int64_t>(a.nslices, 1) + row - 1) / row));
    const int32_t small = daso::small_buckets(ranges, g, small_average);
    const hipError_t e = small > 0 ? daso::launch_buckets(mode, with_stats, a, small, stream)
                                   : daso::launch_step(mode, with_stats, a, grid, lds, stream);
    if (e != hipSuccess) return DASO_EHIP;
    partials = partials || small == 0;
    i += whole ? g.count : 0;
    from = whole ? -1 : g.hi;
    if (!with_stats || a.done != nullptr) continue;
    if (cut.pass_each ? small == 0 : i == ranges.size() && partials) {
      const int32_t buckets = cut.pass_each ? g.count : ranges.size();
      if (daso::launch_stats(a.partials, table, stats, buckets, stream) != hipSuccess) return DASO_EHIP;
    }
    if (!cut.pass_each) {
      a.table += g.count;
      a.slot0 += daso::launch_slots(g, shift);
    }
  }
  return DASO_OK;
}

// A long bucket table is sorted in host memory: running out of it must not
// leave the C entry points as an exception.
int run_groups(daso::Mode mode, StepArgs& a, const daso_bucket* b, int32_t nb,
               daso_bucket_stats* stats, hipStream_t stream, Space space = Space::kAllocated) {
  try {
    return launch_groups(mode, a, b, nb, stats, stream, space);
  } catch (const std::bad_alloc&) {
    return DASO_EHIP;
  }
}

}  // namespace

extern "C" {

int daso_local_avg(const float* const* grads, int32_t g, float* out, int64_t n, hipStream_t stream) {
  const int rc = daso::host::check_local_avg(grads, g, out, n);
  if (rc != DASO_OK || n == 0) return rc;
  StepArgs a;
  memset(&a, 0, sizeof(a));
  for (int32_t r = 0; r < g; ++r) a.grads[r] = grads[r];
  a.g = g;
  a.gavg = out;
  const daso_bucket whole = {0, n, 0, 0};
  return run_groups(daso::kModeAvg, a, &whole, 1, nullptr, stream);
}

int daso_pack_bf16(const float* src, uint16_t* wire, int64_t n, hipStream_t stream) {
  const int rc = daso::host::check_pack(src, wire, n);
  if (rc != DASO_OK || n == 0) return rc;
  StepArgs a;
  memset(&a, 0, sizeof(a));
  a.src = src;
  a.wire = wire;
  const daso_bucket whole = {0, n, 0, 0};
  return run_groups(daso::kModePack, a, &whole, 1, nullptr, stream);
}

}  // extern "C"

namespace {

// Eq. (1) merge with copies and wire of `esz` bytes per element (2: bf16, 4: fp32).
int merge_impl(float* params, const void* const* stale, int32_t P, const daso_bucket* buckets, int32_t nbuckets,
               void* wire, int64_t n, size_t esz, hipStream_t stream) {
  const int rc = daso::host::check_merge(params, stale, P, buckets, nbuckets, wire, n, esz);
  if (rc != DASO_OK || n == 0) return rc;
  StepArgs a;
  memset(&a, 0, sizeof(a));
  for (int32_t i = 0; i < P; ++i) a.stale[i] = stale[i];
  a.P = P;
  a.x = params;
  a.wire = wire;
  a.xf32 = esz == 4 ? 1 : 0;
  return run_groups(daso::kModeMerge, a, buckets, nbuckets, nullptr, stream);
}

}  // namespace

extern "C" {

int daso_global_merge(float* params, const uint16_t* const* stale, int32_t P, const daso_bucket* buckets,
                      int32_t nbuckets, uint16_t* wire, int64_t n, hipStream_t stream) {
  return merge_impl(params, reinterpret_cast<const void* const*>(stale), P, buckets, nbuckets, wire, n, 2, stream);
}

int daso_global_merge_f32(float* params, const float* const* stale, int32_t P, const daso_bucket* buckets,
                          int32_t nbuckets, float* wire, int64_t n, hipStream_t stream) {
  return merge_impl(params, reinterpret_cast<const void* const*>(stale), P, buckets, nbuckets, wire, n, 4, stream);
}

}  // extern "C"

namespace {

// Checks a fused call and fills the kernel arguments that do not depend on the
// launch (streams, counts, constants).  With n == 0 only the counts and the
// exchange type are filled: no pointer is looked at.
int fused_args(const daso_sync_args* args, StepArgs& a) {
  if (args == nullptr) return DASO_EINVAL;
  const daso_sync_args& s = *args;
  daso::host::FusedView v;
  const int rc = daso::host::check_fused(s, &v);
  if (rc != DASO_OK) return rc;
  memset(&a, 0, sizeof(a));
  a.g = s.g;
  a.P = s.P;
  a.xf32 = (s.flags & DASO_EXCHANGE_F32) ? 1 : 0;
  if (s.n == 0) return DASO_OK;
  for (int32_t r = 0; r < s.g; ++r) a.grads[r] = s.grads[r];
  for (int32_t i = 0; i < s.P; ++i) a.stale[i] = v.stale[i];
  a.x = s.params;
  a.m = s.momentum;
  a.wire = v.wire;
  a.gavg = s.grad_avg;
  a.lr = s.lr;
  a.mu = s.mu;
  a.wd = s.weight_decay;
  a.flags = s.flags;
  return DASO_OK;
}

int fused_impl(const daso_sync_args* args, hipStream_t stream, Space space) {
  StepArgs a;
  const int rc = fused_args(args, a);
  if (rc != DASO_OK || args->n == 0) return rc;
  return run_groups(daso::kModeFused, a, args->buckets, args->nbuckets, args->stats, stream, space);
}

}  // namespace

extern "C" {

int daso_fused_sync_step(const daso_sync_args* args, hipStream_t stream) {
  return fused_impl(args, stream, Space::kAllocated);
}

int daso_fused_sync_step_noalloc(const daso_sync_args* args, hipStream_t stream) {
  return fused_impl(args, stream, Space::kFixed);
}

int daso_fused_launch_config(const daso_sync_args* args, daso_launch_config* out) {
  if (out == nullptr) return DASO_EINVAL;
  StepArgs a;
  const int rc = fused_args(args, a);
  if (rc != DASO_OK) return rc;
  const int64_t tile = daso::plan_tile(daso::kModeFused, a.g, a.P, a.xf32 != 0);
  const int64_t ntiles = args->n > 0 ? daso::plan_tiles(args->buckets, args->nbuckets, 0, tile) : 0;
  const int streams = a.g + a.P + 4 + (a.wire ? 1 : 0) + (a.gavg ? 1 : 0);
  const int64_t run = fused_run_elems_override(), cap = fused_cap_override();
  out->tile_elems = tile;
  out->ntiles = ntiles;
  out->xcd_run_tiles = daso::plan_run(streams, std::max<int64_t>(ntiles, 1));
  if (run >= 0 && streams >= daso::kPlanRunStreams)
    out->xcd_run_tiles = static_cast<int32_t>(std::max<int64_t>(1, run / tile));
  out->lds_bytes = daso::lds_for_workgroups_per_cu(streams >= daso::kPlanCapStreams ? 2 : 0);
  if (cap >= 0) out->lds_bytes = daso::lds_for_workgroups_per_cu(static_cast<int32_t>(cap));
  return DASO_OK;
}

}  // extern "C"
