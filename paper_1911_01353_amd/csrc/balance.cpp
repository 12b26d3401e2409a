// Templates per workgroup of an FFT launch, by the size of the launch.
#include "balance.h"

#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

namespace jerk {
namespace {

constexpr double kForward = 1.5;  // a tile's forward transform, in templates
// The tiles of a launch do not keep step: sizes are ranked by the finishing time and this share of the
// largest tile. Over 134 searches and candidate passes whose blocks had changed, that came nearest to
// the measured times (6.8% RMS; 8.2% without it). Gains of 2% and more on that scale were hardly ever losses.
constexpr double kSpread = 0.2;
constexpr double kGain = 0.98;

int32_t blocks_of(const BalanceRun& r) { return (r.members + r.tpb - 1) / r.tpb; }

// Blocks of at most tpb templates, all of about the same size.
int32_t shared_out(int32_t members, int32_t tpb) {
  const int32_t blocks = (members + tpb - 1) / tpb;
  return (members + blocks - 1) / blocks;
}

struct Size {
  double work = 0.0, most = 0.0;  // sum and largest of the tiles' costs
  int64_t tiles = 0;
};

Size size_of(const BalanceRun* runs, int n) {
  Size s;
  for (int i = 0; i < n; ++i) {
    const BalanceRun& r = runs[i];
    if (r.members <= 0 || r.segs <= 0) continue;
    const int64_t blocks = blocks_of(r);
    s.tiles += r.segs * blocks;
    s.work += (double)r.segs * ((double)r.members + (double)blocks * kForward);
    s.most = std::max(s.most, (double)std::min(r.tpb, r.members) + kForward);
  }
  return s;
}

}  // namespace

double dispatch_time(const BalanceRun* runs, int n, int64_t places, double limit) {
  struct Level {
    double time;
    int64_t places;  // that become free then
  };
  std::vector<Level> at{{0.0, places}};  // ascending; at[head...] is the present state
  size_t head = 0;
  auto run = [&](double cost, int64_t tiles) {
    while (tiles > 0) {
      if (at[head].time + cost >= limit) return false;
      if (tiles >= places && at.back().time - at[head].time <= cost) {
        // no place is done twice before every other is done once: whole rounds
        const int64_t rounds = tiles / places;
        for (size_t i = head; i < at.size(); ++i) at[i].time += (double)rounds * cost;
        tiles -= rounds * places;
        continue;
      }
      const int64_t take = std::min(tiles, at[head].places);
      const double end = at[head].time + cost;
      tiles -= take;
      at[head].places -= take;
      if (at[head].places == 0) ++head;
      size_t i = at.size();
      while (i > head && at[i - 1].time > end) --i;
      if (i > head && at[i - 1].time == end) at[i - 1].places += take;
      else at.insert(at.begin() + (std::ptrdiff_t)i, Level{end, take});
    }
    return true;
  };
  for (int i = 0; i < n; ++i) {
    const BalanceRun& r = runs[i];
    if (r.members <= 0 || r.segs <= 0) continue;
    const int32_t blocks = blocks_of(r);
    if (!run((double)r.tpb + kForward, r.segs * (int64_t)(blocks - 1)) ||
        !run((double)(r.members - (blocks - 1) * r.tpb) + kForward, r.segs))
      return limit;
  }
  return at.back().time;
}

// Large blocks amortise the forward transform, but leave the last workgroups of a launch running
// alone, or a small launch short of workgroups; the default rule of the plan, which sees one whole
// group alone, knows neither. Of the block sizes up to 64, shared out evenly over each run's templates,
// the one is taken with which the launch ends first. Row peaks of 101 templates (zmax 100, no jerk
// axis) over 633800 bins: 313 us with the plan's blocks, 252 so; 154 templates' plane over 74788 bins 58.5 and
// 50.6; over 110 launches drawn at random 3.6% less. An estimate in whole rounds of the largest
// block, which no launch keeps to, gained 2.5% and made 6 of them slower, the worst by 25%.
// Where runs stand for several jobs, the dispatch is an estimate; there a size also has to win with
// its largest tile alone at the end, in whatever order the tiles come.
void balance_blocks(BalanceRun* runs, int n, int64_t places, int64_t max_tiles, bool whole) {
  bool any = false;
  for (int i = 0; i < n; ++i) any = any || (runs[i].free && runs[i].members > 0);
  if (!any) return;
  const Size own = size_of(runs, n);
  if (own.tiles <= places) return;  // one round: the plan's rule spreads it over the device
  const double own_time = dispatch_time(runs, n, places, std::numeric_limits<double>::infinity());
  double best = kGain * (own_time + kSpread * own.most);
  int32_t size = 0;
  std::vector<BalanceRun> r(runs, runs + n);
  for (int32_t tpb : {64, 56, 48, 40, 32, 28, 24, 20, 16, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2}) {
    for (int i = 0; i < n; ++i)
      if (r[i].free && r[i].members > 0) r[i].tpb = shared_out(r[i].members, tpb);
    const Size s = size_of(r.data(), n);
    if (s.tiles > max_tiles) break;  // smaller blocks only add workgroups
    const double least = s.work / (double)places;
    const double limit = std::min(own_time, best - kSpread * s.most);
    if (std::max(least, s.most) >= limit || (!whole && least + s.most >= own_time)) continue;
    const double time = dispatch_time(r.data(), n, places, limit);
    if (time < limit) {
      best = time + kSpread * s.most;
      size = tpb;
    }
  }
  if (size == 0) return;
  for (int i = 0; i < n; ++i)
    if (runs[i].free && runs[i].members > 0) runs[i].tpb = shared_out(runs[i].members, size);
}

// The filter of a candidate pass reads a tile's hits one after the other, a thread per tile, at about
// 0.3 us a hit. Larger tiles hold more of them: with the staging level at 2 mean powers, blocks of 16
// templates grown to 28 and 60 made the filter most of the search (765 templates over 2^18 bins 5.2 -> 10.2 ms),
// at 5.4 mean powers they took 1.82 ms instead of 1.50. So only where a larger tile expects at most 16 hits
// (5 us; at the usual levels above 11 mean powers it expects one or two).
bool candidate_blocks_allowed(int32_t tpb, int32_t own, int32_t U, double pre) {
  return tpb <= own || 2.0 * (double)tpb * (double)U * std::exp(-std::max(0.0, pre)) <= 16.0;
}

}  // namespace jerk
