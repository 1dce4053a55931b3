// The cut of a call into launches (daso_plan.h) against its rules on random bucket
// tables: every element in exactly one range with its own bucket's staleness, launches
// that follow each other, partials that never share a place and stay within the
// launch's.  Exit status 0 when every expectation holds.
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "daso_plan.h"

static int failures = 0;
#define EXPECT(cond)                                                                   \
  do {                                                                                 \
    if (!(cond)) {                                                                     \
      if (++failures < 20) std::fprintf(stderr, "line %d: %s\n", __LINE__, #cond);     \
    }                                                                                  \
  } while (0)

int main() {
  std::mt19937_64 rng(11);
  for (int trial = 0; trial < 4000; ++trial) {
    // a table tiling [0, n), some buckets empty, in random, ascending or descending order
    const int64_t n = 1 + static_cast<int64_t>(rng() % (trial % 4 == 0 ? 300000 : 30000));
    const int want_nb = 1 + static_cast<int>(rng() % (trial % 3 == 0 ? 400 : 12));
    std::set<int64_t> cuts = {0, n};
    while (static_cast<int>(cuts.size()) < want_nb + 1 && static_cast<int64_t>(cuts.size()) <= n)
      cuts.insert(rng() % 2 ? static_cast<int64_t>(rng() % n) : (static_cast<int64_t>(rng() % n) >> 8) << 8);
    std::vector<daso_bucket> b;
    for (auto it = cuts.begin(); std::next(it) != cuts.end(); ++it) {
      b.push_back({*it, *std::next(it) - *it, static_cast<int32_t>(rng() % 3), 0});
      if (rng() % 6 == 0) b.push_back({*it, 0, static_cast<int32_t>(rng() % 3), 0});
    }
    if (trial % 3 == 1) std::reverse(b.begin(), b.end());
    if (trial % 3 == 2) std::shuffle(b.begin(), b.end(), rng);
    std::vector<int32_t> S(static_cast<size_t>(n), -1);
    for (const auto& k : b)
      for (int64_t e = k.start; e < k.start + k.numel; ++e) S[static_cast<size_t>(e)] = k.S;
    for (const bool with_stats : {false, true}) {
      const daso::Ranges r(b.data(), static_cast<int32_t>(b.size()), with_stats);
      EXPECT(!with_stats || r.size() == static_cast<int32_t>(b.size()));
      int64_t pos = 0;
      std::set<int32_t> outs;
      for (int32_t i = 0; i < r.size(); ++i) {
        EXPECT(r[i].start == pos);
        for (int64_t e = r[i].start; e < r[i].end; ++e) EXPECT(S[static_cast<size_t>(e)] == r[i].S);
        pos = r[i].end;
        if (with_stats) {
          outs.insert(r[i].out);
          const daso_bucket& k = b[static_cast<size_t>(r[i].out)];
          EXPECT(k.start == r[i].start && k.start + k.numel == r[i].end && k.S == r[i].S);
        } else {
          EXPECT(r[i].end > r[i].start);
          EXPECT(i == 0 || r[i - 1].S != r[i].S);
        }
      }
      EXPECT(pos == n);
      EXPECT(!with_stats || outs.size() == b.size());
      for (const int waves : {1, 4, 8}) {
        const int shift = daso::super_shift(waves);
        const int64_t room = rng() % 2 ? INT64_MAX : 8 * static_cast<int64_t>(8 + rng() % 40);
        int64_t hi = 0;
        for (int32_t i = 0; i < r.size();) {
          const daso::Group g = daso::group_at(r, i, shift, room);
          EXPECT(g.first == i && g.count >= 1 && g.count <= daso::kLaunchBuckets);
          EXPECT(g.lo == hi && g.lo == r[i].start && g.hi == r[i + g.count - 1].end);
          EXPECT(g.count == 1 || daso::launch_slots(g, shift) <= room);
          hi = g.hi;
          // the places that a launch's workgroups write: bucket k in each superblock it lies in
          const int64_t sb0 = g.lo >> shift;
          std::set<int64_t> places;
          for (int32_t k = 0; k < g.count; ++k) {
            if (r[i + k].end == r[i + k].start) continue;
            for (int64_t sb = r[i + k].start >> shift; sb <= (r[i + k].end - 1) >> shift; ++sb) {
              const int64_t slot = daso::slot_of(sb - sb0, k);
              EXPECT(slot >= 0 && slot + 8 <= daso::launch_slots(g, shift));
              EXPECT(places.insert(slot).second);
            }
          }
          i += g.count;
        }
        EXPECT(hi == n);
        // with a range cut wherever its partials alone exceed the room
        int64_t end = 0, from = -1;
        for (int32_t i = 0; i < r.size();) {
          const daso::Group g = daso::cut_to(daso::group_at(r, i, shift, room, from), shift, room);
          EXPECT(g.first == i && g.lo == end && daso::launch_slots(g, shift) <= room);
          const bool whole = g.hi == r[i + g.count - 1].end;
          EXPECT(whole || (g.count == 1 && g.hi > g.lo && g.hi < r[i].end && g.hi % (int64_t(1) << shift) == 0));
          end = g.hi;
          i += whole ? g.count : 0;
          from = whole ? -1 : g.hi;
        }
        EXPECT(end == n);
      }
    }
  }
  // The fixed scratch of the no-alloc entry point, with more buckets than its table could
  // list, the largest bucket that its limit lets pass, or both: every launch's table
  // and partials stay within it.
  const int64_t scratch = static_cast<int64_t>(DASO_NOALLOC_SCRATCH_BYTES) - 256;
  const int64_t big = (static_cast<int64_t>(DASO_NOALLOC_SCRATCH_BYTES) - 256 - 260) / 24 * 2048;
  for (const int64_t large : {int64_t(1), big})
    for (const int64_t lead : {int64_t(0), int64_t(2047)})
      for (const int32_t nb : {1, 63, 130, 1100, 2700, 3000, 100000, 1500000}) {
        std::vector<daso_bucket> b;
        int64_t pos = 0;
        if (lead > 0) b.push_back({0, lead, 1, 0}), pos = lead;
        b.push_back({pos, large - (large > lead ? lead : 0), 2, 0});
        pos += b.back().numel;
        while (static_cast<int32_t>(b.size()) < nb) b.push_back({pos++, 1, 1, 0});
        const daso::Ranges r(b.data(), static_cast<int32_t>(b.size()), true);
        for (const int waves : {4, 8}) {
          const int shift = daso::super_shift(waves);
          const daso::Cut c = daso::cut_of(r, shift, true, scratch);
          int64_t slots = 0, most = 0, from = -1;
          for (int32_t i = 0; i < r.size();) {
            const daso::Group g = daso::cut_to(daso::group_at(r, i, shift, c.room, from), shift, c.room);
            const bool whole = g.hi == r[i + g.count - 1].end;
            most = std::max(most, daso::launch_slots(g, shift));
            slots += daso::launch_slots(g, shift);
            EXPECT(g.count <= c.table && (whole || c.pass_each));
            i += whole ? g.count : 0;
            from = whole ? -1 : g.hi;
          }
          EXPECT(c.pass_each || (c.table == r.size() && slots == c.slots));
          EXPECT(c.table * daso::kEntryBytes + (c.pass_each ? most : slots) * daso::kPartialBytes <= scratch);
        }
      }
  if (failures == 0) std::puts("plan checks ok");
  return failures == 0 ? 0 : 1;
}
