// How many pages a wave of an attention workgroup walks (host; plain C++).
#pragma once

#include <algorithm>

namespace laser {

constexpr int kLongestRun = 256;  // pages per wave
constexpr int kXcds = 8;
constexpr int kFewItems = 4 * kXcds;  // work items per kv head, below which the XCDs' shares have to be even
constexpr int kMidRun = 8;            // pages per wave where one round of workgroups is out of reach

struct RunGroup {
  int pages, tiles;  // pages of a row group, its query tiles (work items per split)
};

// Pages per wave of a forward of up to 64 rows, at least `base`.  A workgroup (waves waves) keeps its
// pages streaming, so one round of long runs, every workgroup resident at once, beats several rounds of
// short ones, each with its own start-up and partials (8 KV heads, batch 8, 68k positions: 63.5 us with
// runs of at most 4 pages, 52.9 with one round), and a last round that is nearly empty costs most (runs
// of 16 pages: 1.4 rounds, the step 840 against 800 us).  That holds where the round is even:
// - a run stays within twice a wave's even share of all pages.  One long request among many short ones
//   cannot be spread over a round that the short ones' workgroups fill; lengthening only strings its
//   pages on a few waves (8 KV heads, 63 requests of 100 positions and one of 14,000, two layers: 520 us
//   with runs of 110 pages, 361 with 8, 357 with 4);
// - a head's items are kFewItems or more, or fill the XCDs evenly (as many items on each, 90% as long as
//   the longest on the average).  Workgroups of one item run on one XCD (item i on XCD i mod 8), so few
//   items of several lengths load them unevenly (two layers of 32 KV heads, head dim 64, a round and runs
//   of at most 8 pages: 16 requests of 100-4,000 positions 222 us and 205, 24 of those 302 and 257, 5 of
//   8,000 in 20 items 234 and 216; but 16 of 8,000 437 and 480, 24 of 3,000 306 and 327, 24 of 14,000 in
//   runs of 219 pages 938 and 1,039).
// Groups that are more than one round even when each is one workgroup are left so if they are alike
// (32 KV heads, 24 requests of 3,000 positions: 604 us, 631 with runs of 8 pages; not 40 requests of
// 100-4,000: 810 against 745).  Elsewhere: half an even share, at most kMidRun pages (32 KV heads, batch
// 16, 1,000-14,000: 953 us at 4 pages, 910 at 8; batch 64, 14,000 and 63 x 1,000 positions: 777 against 755).
inline int run_pages(const RunGroup* g, int n, int heads, int waves, int resident, int base) {
  long long units = 0, tiles = 0;
  int most = 0;  // pages of the longest group
  for (int i = 0; i < n; ++i) {
    units += (long long)g[i].pages * g[i].tiles;
    tiles += g[i].tiles;
    most = std::max(most, g[i].pages);
  }
  auto items = [&](int b) {
    long long k = 0;
    for (int i = 0; i < n; ++i) k += (long long)((g[i].pages + waves * b - 1) / (waves * b)) * g[i].tiles;
    return k;
  };
  if (items(base) * heads <= resident) return base;
  const long long share = units * heads / ((long long)waves * resident);  // pages per resident wave
  if (tiles * heads <= resident) {
    const int longest = (int)std::min<long long>(kLongestRun, 2 * share + 1);
    for (int b = base + 1; b <= longest; ++b) {
      const long long k = items(b);
      if (k * heads > resident) continue;
      if (k >= kFewItems) return b;
      int longest_item = 0;
      for (int i = 0; i < n; ++i) {
        const int w = (g[i].pages + waves * b - 1) / (waves * b);
        if (w) longest_item = std::max(longest_item, (g[i].pages + w - 1) / w);
      }
      if (10 * units >= 9 * ((k + kXcds - 1) / kXcds * kXcds) * longest_item) return b;
      break;
    }
  } else {
    const int whole = (most + waves - 1) / waves;  // every group one workgroup
    if (tiles >= 3 * kXcds && whole <= kLongestRun && 4ll * most * tiles <= 5 * units) return std::max(base, whole);
  }
  return (int)std::max<long long>(base, std::min<long long>(kMidRun, share / 2));
}

}  // namespace laser
