// How a launch of the FFT kernels shares its templates out over workgroups: host arithmetic on
// counts alone (no HIP), so that it can be checked without a device.
#pragma once
#include <cstdint>

namespace jerk {

// The tiles of one job, or of several of one width group: `segs` segments times blocks of at most
// `tpb` of `members` templates, block after block.
struct BalanceRun {
  int64_t segs;
  int32_t members;
  int32_t tpb;
  bool free;  // tpb may be changed
};

// Finishing time of the runs' tiles when each goes, in order, to the place that is free first: in
// templates, a tile costing its templates and the forward transform. Gives up, with a value not
// below `limit`, once it knows that it will not end earlier.
double dispatch_time(const BalanceRun* runs, int n, int64_t places, double limit);

// Changes the runs' tpb (those that are free) where the launch then ends clearly earlier on
// `places` workgroups at a time. whole: the runs are the launch's jobs in order; otherwise some stand
// for several jobs whose tiles are mixed. Never more than max_tiles tiles. Only speed depends on it.
void balance_blocks(BalanceRun* runs, int n, int64_t places, int64_t max_tiles, bool whole);

// Whether a candidate pass, whose staged hits are read back tile by tile, may take blocks of `tpb`
// templates instead of the plan's `own`. U: lags of a segment, pre: the staging level.
bool candidate_blocks_allowed(int32_t tpb, int32_t own, int32_t U, double pre);

}  // namespace jerk
