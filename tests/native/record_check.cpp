// The cursor protocol of the deposit records, on the CPU: the words and
// constants of ctd_records.h and the steps the kernel follows with them.
// Reads "seed lanes deposits segments start high" lines from stdin: `lanes`
// lanes make `deposits` deposits each into one bucket whose cursor starts as a
// full segment 1 with count `start` (1 taken as kLogSeg), with `segments` more
// segments; `high` is the count from which a deposit winds the word back (0:
// never).  Lanes take turns at random, one memory operation a turn.  Prints
// "ok", or the first violation: a record outside the bucket's segments, two
// records in one place, a deposit lost, a segment number that nobody installed.
#include <cstdint>
#include <cstdio>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "ctd_records.h"

namespace {

struct Rng {
  uint64_t s;
  uint32_t next() {
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)(s >> 33);
  }
};

enum Step { kAdd, kSegment, kWind, kInstall, kAgain };
struct Lane {
  Step step = kAdd;
  uint64_t left = 0, w = 0;
  uint32_t next = 0;
  int t = 0;
};

std::string play(uint64_t seed, int lanes, uint64_t deposits, uint32_t segments, uint64_t start,
                 uint64_t high) {
  using ctd::kLogSeg;
  const uint32_t first = 2, end = first + segments;
  uint64_t cur = (uint64_t)1 << 32 | start;
  uint32_t seg_next = first;
  std::set<uint32_t> known{1};
  std::set<uint64_t> places;
  uint64_t tally = 0, records = 0;
  std::vector<Lane> lane((size_t)lanes);
  for (Lane &l : lane) l.left = deposits;
  Rng rng{seed};
  int live = lanes;
  while (live > 0) {
    Lane &l = lane[rng.next() % (uint32_t)lanes];
    if (l.left == 0) continue;
    bool done = false, record = false;
    const uint32_t count = (uint32_t)l.w;
    switch (l.step) {
      case kAdd:
      case kAgain:
        l.w = cur++;
        if (!known.count((uint32_t)(l.w >> 32))) return "a segment nobody installed";
        if ((uint32_t)l.w < kLogSeg) done = record = true;
        else if (l.step == kAdd) l.t = 0, l.step = kSegment;
        else ++l.t, l.step = kSegment;
        break;
      case kSegment: {
        const bool mine = count == kLogSeg;
        l.next = seg_next;
        if (mine) ++seg_next;
        if (l.next >= end || (!mine && l.t >= 16)) {
          if (high && count >= high) l.step = kWind;
          else ++tally, done = true;
        } else if (mine) {
          l.step = kInstall;
        } else {
          l.step = kAgain;
        }
        break;
      }
      case kWind:
        if (cur == l.w + 1) cur = ctd::cursor_full(l.w);
        ++tally;
        done = true;
        break;
      case kInstall:
        known.insert(l.next);
        l.w = (uint64_t)l.next << 32;
        cur = l.w | 1u;
        done = record = true;
        break;
    }
    if (!done) continue;
    if (record) {
      const uint32_t seg = (uint32_t)(l.w >> 32);
      if (seg < first || seg >= end || (uint32_t)l.w >= kLogSeg) return "a record out of place";
      if (!places.insert((uint64_t)seg * kLogSeg + (uint32_t)l.w).second) return "a place taken twice";
      ++records;
    }
    l.step = kAdd;
    if (--l.left == 0) --live;
  }
  if (records + tally != deposits * (uint64_t)lanes) return "deposits lost";
  if ((uint32_t)(cur >> 32) != (segments ? end - 1 : 1u)) return "a segment nobody installed";
  return "ok";
}

}  // namespace

int main() {
  unsigned long long seed, deposits, start, high;
  int lanes;
  unsigned segments;
  while (std::scanf("%llu %d %llu %u %llu %llu", &seed, &lanes, &deposits, &segments, &start,
                    &high) == 6)
    std::printf("%s\n",
                play(seed, lanes, deposits, segments, start == 1 ? ctd::kLogSeg : start, high)
                    .c_str());
  return 0;
}
