// Internal interface between the C-ABI entry points (daso_api.hip) and the
// kernels (daso_kernels.hip).  Not part of the public ABI.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

#include "daso.h"
#include "daso_plan.h"

namespace daso {

constexpr int kStatsBlock = 1024;  // threads of stats_kernel
constexpr int kRowShift = 20;      // at most 2^20 workgroups in a row of a launch's grid

// Occupancy.  A wavefront has all its loads in flight at once, and beyond some number of them
// per CU more only spread the front over more DRAM pages: by instance 50 to 110 KB for
// workgroups of one wavefront, 50 to 160 KB for those of four, 180 to 260 KB for those of
// eight.  Each workgroup therefore holds LDS that it does not use, which caps how many share
// a CU (lds_of in daso_api.hip states the rule, with the counts on either side).
constexpr int32_t kCuLdsBytes = 160 * 1024;  // LDS per CU on gfx950

// LDS per workgroup that lets at most k workgroups share a CU: a 1 KB margin
// covers the kernel's own few bytes of LDS and the allocation granule.
inline int32_t lds_for_workgroups_per_cu(int32_t k) { return k >= 1 ? kCuLdsBytes / k - 1024 : 0; }

// Elements up to which a call is short: its launches are over before the front of their workgroups
// has spread, so it takes no occupancy cap (lds_of) and no workgroups of eight wavefronts (with_waves).
constexpr int64_t kShortCall = int64_t(3) << 20;

// An eager fused launch with statistics of at most this many wavefronts (131,072
// parameters) has its last workgroup sum the statistics (StepArgs::done) instead of
// a second launch.  The workgroups count themselves done in one counter, at 5 to 11 ns
// each one after the other: 65,536 parameters (g = 4, P = 2) take 5.2 us against 8.2 in
// two launches, 200,000 (g = 4, P = 8) 8.0 against 8.2, 300,000 9.7 against 8.2, 2M 35
// against 20.5.  Captured calls keep the second launch, whose host cost a graph replay does not pay.
constexpr int64_t kFinishStatsMaxWaves = 512;

// Bytes at the start of a statistics scratch buffer that hold the counter of
// StepArgs::done (zero whenever no launch is running); the bucket table and the
// partials follow.
constexpr size_t kStatsCounterBytes = 256;

// Side-output partial of one bucket and slice, reduced per bucket by stats_kernel.
struct SlicePartial {
  double grad_sq;
  double delta_sq;
  uint64_t nonfinite;
};

// Where stats_kernel finds the partials of a bucket and puts its statistics.
struct BucketSlots {
  int64_t first, end;
  int32_t out;
  int32_t add;  // nonzero: the launch before had the bucket's first elements, whose statistics these are added to
};

// Kernel arguments, passed by value (3.7 KB).
struct StepArgs {
  const float* grads[DASO_MAX_G];
  const void* stale[DASO_MAX_P];  // bf16 patterns, or fp32 when xf32
  float* x;              // params (merge, mean, fused: in place)
  float* m;              // momentum (fused, in place)
  int64_t lo, hi;        // the launch's elements
  int64_t sb0;           // first superblock of the launch
  int64_t nslices;       // its workgroups with work: 8 per superblock that it overlaps
  const float* src;      // pack: source fp32
  void* wire;            // packed output (bf16, or fp32 when xf32) or nullptr
  float* gavg;           // local average output or nullptr
  SlicePartial* partials;  // (stats only) of the call, see slot_of
  BucketSlots* table;    // (stats only) nb entries written by workgroup 0 for stats_kernel
  int64_t slot0;         // (stats only) the launch's first partial
  daso_bucket_stats* stats;  // per-bucket outputs (stats only), in the caller's order
  uint32_t* done;        // (stats only) nonnull: no stats_kernel; the workgroup that finishes last
                         // sums the statistics.  A counter that is zero before the launch and
                         // that the launch leaves at zero.
  int32_t g;
  int32_t P;
  float lr;
  float mu;
  float wd;
  float g_inv;           // 1 / g, rounded to nearest
  uint32_t flags;
  int32_t xf32;          // nonzero: fp32 exchange (stale copies and wire are fp32)
  int32_t nb;            // buckets in this launch
  int32_t cont;          // nonzero: the first of them began in the launch before (BucketSlots::add)
  int64_t start[kLaunchBuckets + 1];  // the buckets, sorted and back to back: bucket i is [start[i], start[i + 1])
  int32_t S[kLaunchBuckets];          // staleness of Eq. (1)
  float inv[kLaunchBuckets];          // 1 / (2S + P), rounded to nearest (0 when 2S + P is 0)
  int32_t out[kLaunchBuckets];        // (stats only) index in the caller's table
  int64_t n;             // elements of the call's buffers
  int32_t in_place_avg;  // nonzero: gavg is one of the grads
};

// Arguments of stats_kernel, kept to a few pointers: the host cost of a launch
// grows with the size of its arguments (about 2.7 us with 16 bytes, 4 us with
// 2.7 KB on MI355X), and what it needs of each bucket is in the table.
struct StatsArgs {
  const SlicePartial* partials;
  const BucketSlots* table;
  daso_bucket_stats* stats;
};

// The instance that runs `mode` with these arguments: wavefronts per workgroup, and
// whether its stream counts are fixed at compile time, bounded there, or neither.
enum class Counts { kExact, kBounded, kUnbounded };
struct Shape {
  int waves;
  Counts counts;
};
Shape launch_shape(Mode mode, bool with_stats, const StepArgs& args);

// Enqueue one launch of `mode` over the buckets in `args` on `grid` workgroups (one
// per slice, in rows of 2^kRowShift), each holding `lds` bytes of LDS besides the kernel's own.
hipError_t launch_step(Mode mode, bool with_stats, const StepArgs& args, dim3 grid, uint32_t lds,
                       hipStream_t stream);

// Enqueue one launch of `mode` (fused, merge) over the buckets in `args`, all small: `waves`
// wavefronts for each, or with statistics a workgroup, which writes them itself.
hipError_t launch_buckets(Mode mode, bool with_stats, const StepArgs& args, int32_t waves, hipStream_t stream);

// Enqueue the sums of the statistics of `nb` buckets, whose launches wrote `table` and `partials`.
hipError_t launch_stats(const SlicePartial* partials, const BucketSlots* table, daso_bucket_stats* stats,
                        int32_t nb, hipStream_t stream);

// Enqueue the zeroing of the counter at the start of a new statistics buffer.
hipError_t clear_stats_counter(void* buffer, hipStream_t stream);

}  // namespace daso
