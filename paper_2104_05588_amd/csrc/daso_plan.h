// How a call is cut into launches and its elements dealt to workgroups: host-only
// code and constants, shared with the kernels and compiled on its own in the tests.
// Not part of the public ABI.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "daso.h"

namespace daso {

// kModeMean is kModeMerge with S = 0 for every element: the plain average of the
// copies, which does not read the parameters it replaces.
enum Mode : int { kModeAvg = 0, kModePack = 1, kModeMerge = 2, kModeFused = 3, kModeMean = 4 };

// Work decomposition.  A wavefront takes one piece of kPiece = 256 consecutive
// elements, 4 per lane.  Pieces go to workgroups by superblock: the 8 workgroups
// 8k .. 8k + 7 of a launch share superblock k, of which workgroup s takes the
// pieces s, s + 8, s + 16, ... (one per wavefront).  Workgroups are dispatched to the 8
// XCDs in turn, so each XCD reads and writes every eighth 1 KB of an fp32 stream
// (512 B of a bf16 one) and the chip sweeps the streams front to back with a
// front of a few hundred KB per stream.  Superblocks are counted from element 0
// of the buffers, so a wavefront's accesses are whole cache lines wherever a bucket
// begins.
//
// Measured on MI355X with bare copies of 1 GiB (no arithmetic): dealing 4 KB
// or 1 KB to the XCDs in turn moves 6.5 to 6.7 TB/s, 8 KB or 16 KB 5.9 to 6.3, runs
// of 64 KB 5.1 to 5.4 (the loss is in the writes: reads alone reach 7.0 TB/s in any order);
// and a wavefront that takes one piece and ends, leaving the order to the
// dispatcher, beats one that walks over several (4 or 16 pieces: 10 to 20% slower),
// prefetching the next or not.
constexpr int kVec = 4;            // consecutive elements per lane
constexpr int kPiece = 64 * kVec;  // elements per wavefront
// A superblock of 8 workgroups of `waves` wavefronts (1, 4 or 8) holds 8 * waves pieces.
constexpr int super_shift(int waves) { return waves == 1 ? 11 : waves == 4 ? 13 : 14; }
static_assert(int64_t(1) << super_shift(1) == 8 * kPiece && int64_t(1) << super_shift(4) == 8 * 4 * kPiece &&
                  int64_t(1) << super_shift(8) == 8 * 8 * kPiece,
              "a superblock is the pieces of 8 workgroups");

constexpr int kLaunchBuckets = 128;

// Partials of a launch, by bucket and superblock: bucket i (of those sorted by
// start) has 8, one per workgroup, for each superblock it overlaps.  Two neighbours may
// share a superblock, so bucket i's begin i superblocks late, which keeps them apart.
// `sb` is a superblock counted from the launch's first.
constexpr int64_t slot_of(int64_t sb, int i) { return (sb + i) * 8; }

// The caller's buckets in order of their start (empty ones first among equals).
// Without statistics only their staleness matters: empty buckets are left out
// and neighbours of one staleness become one, so that a table of any length with one
// S, as the driver passes, is a single launch.
struct Range {
  int64_t start, end;
  int32_t S;
  int32_t out;  // index in the caller's table
};

class Ranges {
 public:
  Ranges(const daso_bucket* b, int32_t nb, bool with_stats) {
    if (nb > kFew) many_.resize(static_cast<size_t>(nb));
    r_ = nb > kFew ? many_.data() : few_;
    const bool back = nb > 1 && b[0].start > b[nb - 1].start;  // plans list buckets from the last to the first
    for (int32_t i = 0; i < nb; ++i) {
      const int32_t k = back ? nb - 1 - i : i;
      if (b[k].numel > 0 || with_stats) r_[n_++] = Range{b[k].start, b[k].start + b[k].numel, b[k].S, k};
    }
    const auto before = [](const Range& x, const Range& y) {
      return x.start != y.start ? x.start < y.start : x.end < y.end;
    };
    if (!std::is_sorted(r_, r_ + n_, before)) std::sort(r_, r_ + n_, before);
    if (with_stats) return;
    int32_t kept = 0;
    for (int32_t i = 1; i < n_; ++i) {
      if (r_[i].S == r_[kept].S) r_[kept].end = r_[i].end;
      else r_[++kept] = r_[i];
    }
    n_ = kept + 1;
  }
  Ranges(const Ranges&) = delete;
  Ranges& operator=(const Ranges&) = delete;
  int32_t size() const { return n_; }
  const Range& operator[](int32_t i) const { return r_[i]; }

 private:
  static constexpr int32_t kFew = 64;
  Range few_[kFew];
  std::vector<Range> many_;
  Range* r_;
  int32_t n_ = 0;
};

// One launch: `count` ranges from `first`, covering the elements [lo, hi).
struct Group {
  int32_t first, count;
  int64_t lo, hi;
};

// Superblocks that [lo, hi) overlaps.
inline int64_t superblocks(int64_t lo, int64_t hi, int shift) {
  return hi > lo ? ((hi - 1) >> shift) - (lo >> shift) + 1 : 0;
}

// Partials that a launch has places for (slot_of).
inline int64_t launch_slots(const Group& g, int shift) { return 8 * (superblocks(g.lo, g.hi, shift) + g.count); }

// The launch that begins at element `from` (-1: the start) of range `first`.
inline Group group_at(const Ranges& r, int32_t first, int shift, int64_t max_slots, int64_t from = -1) {
  Group g{first, 1, from < 0 ? r[first].start : from, r[first].end};
  while (g.count < kLaunchBuckets && first + g.count < r.size()) {
    const Group more{first, g.count + 1, g.lo, r[first + g.count].end};
    if (launch_slots(more, shift) > max_slots) break;
    g = more;
  }
  return g;
}

// The wavefronts for each bucket of a launch that bucket_kernel takes, as many as the largest
// bucket has pieces; 0 if it does not: its buckets have at most `average` elements on average
// and none more than twice that.
inline int32_t small_buckets(const Ranges& r, const Group& g, int64_t average) {
  if (g.count < 2 || g.hi - g.lo > average * g.count) return 0;
  int64_t most = 1;
  for (int32_t k = g.first; k < g.first + g.count; ++k) most = std::max(most, r[k].end - std::max(r[k].start, g.lo));
  return most > 2 * average ? 0 : static_cast<int32_t>((most + kVec - 2) / kPiece + 1);
}

// A launch of one range whose partials alone are more than max_slots (at least 16), cut at a
// superblock so that they fit: the next launch begins where this one ends.
inline Group cut_to(const Group& g, int shift, int64_t max_slots) {
  if (launch_slots(g, shift) <= max_slots) return g;
  return Group{g.first, 1, g.lo, ((g.lo >> shift) + max_slots / 8 - 1) << shift};
}

// How the statistics of a call lie in a scratch whose first bytes are used: a table of
// `table` entries, then the partials.  When the partials and table
// entries of all launches fit, they share one statistics pass.  Else each launch has
// a pass of its own, reuses the places of the one before and needs a table of kLaunchBuckets
// entries alone; `room` then limits the partials of a launch, and a bucket that has more
// takes several launches (cut_to), whose passes add up its statistics.
constexpr int64_t kPartialBytes = 24, kEntryBytes = 24;

// A call's launches share a pass of at most kPassBuckets buckets: it has a workgroup of 1024
// threads for each, and a dispatch counts its work-items in 32 bits.  In an
// allocated scratch the shared pass may take kSharedBytes more than a call of so many
// elements holds anyway (least_bytes), enough for some 150,000 buckets: beyond, a pass
// each costs some 4 us per 128 buckets, which take 10 to 100 us by themselves, and spares
// 24 to 28 KB for each 128 of them that would be held for good.
constexpr int32_t kPassBuckets = 1 << 20;
constexpr int64_t kSharedBytes = int64_t(32) << 20;

struct Cut {
  bool pass_each;
  int64_t table, room, slots, launches;
};

inline Cut cut_of(const Ranges& r, int shift, bool with_stats, int64_t bytes) {
  Cut c{false, with_stats ? r.size() : 0, INT64_MAX, 0, 0};
  for (int32_t i = 0; i < r.size(); ++c.launches) {
    const Group g = group_at(r, i, shift, c.room);
    c.slots += launch_slots(g, shift);
    i += g.count;
  }
  if (with_stats && (r.size() > kPassBuckets || c.slots > (bytes - c.table * kEntryBytes) / kPartialBytes)) {
    c.pass_each = true;
    c.table = kLaunchBuckets;
    c.room = (bytes - c.table * kEntryBytes) / kPartialBytes;
  }
  return c;
}

// An allocated scratch holds at least what any one launch over n elements needs, also in
// the finest split that takes statistics (4 wavefronts per workgroup): 24 bytes per 1024
// elements and 27 KB.
inline int64_t least_bytes(int64_t n) {
  const int64_t slots = launch_slots(Group{0, kLaunchBuckets, 0, n}, super_shift(4));
  return kLaunchBuckets * kEntryBytes + slots * kPartialBytes;
}

// -------------------------------------------------------------- the tiled plan
// A coarser decomposition of a fused step, which daso_fused_launch_config
// reports for tools that time the same streams and in whose tiles the limit of the
// no-alloc entry point is stated: tiles of 2048 elements of a bucket (1024 when a vector of every
// stream takes more than 48 registers), runs of consecutive tiles per XCD
// from 9 streams (about 64 blocks of 8 runs per launch), and LDS that lets 2 workgroups of a tile
// each share a CU from 10.
constexpr int32_t kPlanBuckets = 64;  // per launch
constexpr int kPlanRunStreams = 9;
constexpr int kPlanCapStreams = 10;

inline int64_t plan_tile(Mode mode, int g, int P, bool xf32) {
  const auto pow2 = [](int k) { return k == 2 || k == 4 || k == 8 || k == 16 || k == 32; };
  if (mode == kModeMerge) return !xf32 && P == 32 ? 1024 : 2048;
  if (mode != kModeFused) return 2048;
  int regs = 0;
  if ((g == 4 || g == 8) && pow2(P)) regs = 4 * g + (xf32 ? 4 : 2) * P + 8;
  else if (xf32) return 2048;
  else if (P == 0 && (g == 1 || g == 2 || g == 4 || g == 8)) regs = 4 * g + 8;
  else if (g <= 4 && P <= 16) regs = 4 * 4 + 2 * (P <= 8 ? 8 : 16) + 8;
  else if (g <= 8 && P <= 16 && (g < 8 || P > 8)) regs = 4 * 8 + 2 * (P <= 8 ? 8 : 16) + 8;
  else return 2048;
  return regs <= 48 ? 2048 : 1024;
}

// Tiles of the plan's launch that starts at bucket i: those of the grid counted from element
// 0 that each bucket overlaps.
inline int64_t plan_tiles(const daso_bucket* b, int32_t nb, int32_t i, int64_t tile) {
  int64_t t = 0;
  for (int32_t k = i; k < std::min(nb, i + kPlanBuckets); ++k)
    if (b[k].numel > 0) t += (b[k].start + b[k].numel - 1) / tile - b[k].start / tile + 1;
  return t;
}

inline int32_t plan_run(int streams, int64_t ntiles) {
  int64_t run = 1;
  if (streams >= kPlanRunStreams)
    while (run * 2 <= ntiles / 512 && run < (int64_t(1) << 20)) run *= 2;
  return static_cast<int32_t>(run);
}

// The scratch of the plan's statistics: a 256-byte counter, 24 bytes per tile, a table of 65 words.
inline size_t plan_scratch(int64_t tiles) {
  return 256 + static_cast<size_t>(tiles) * 24 + (kPlanBuckets + 1) * sizeof(int32_t);
}

}  // namespace daso
