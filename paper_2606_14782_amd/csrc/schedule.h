// The order of a prompt call's stages, and how many copies of a buffer the
// layers in flight need.  Host code without any HIP, so that a CPU test can
// walk the schedule.
#pragma once

namespace bacon {

// Copies of the buffers that pass between the stages of a layer, which the
// layers take in turn (layer l the copy l mod their number).  Iteration i of a
// prompt call writes layer i's budget tables and then runs one launch that
// holds a stage of each of several layers (on larger grids the K passes of
// layer i in launches before it); what a later layer writes must have been
// read by then.
//  * partials, normalisers, V and the pooled vectors, the lists, their counts
//    and records are read by the next stage only: two copies;
//  * B is read until the scores, two stages after pass 2: three;
//  * its histogram is counted by pass 2 and cleared, for the layer that takes
//    the copy next, by the candidate job three stages on: four;
//  * the S keys and histogram are cleared by the calibration and read until
//    the final job: four;
//  * the allocation's pooled scores are read two stages on: three, its
//    histogram cleared three stages on: four;
//  * the budget tables are written ahead of all the layer's stages and read
//    until the last of them.
// The head-wise allocation puts kAllocLag stages between pass 2 and the
// calibration, and B, its histogram and the E history as many copies more.
constexpr int kAllocLag = 3;
constexpr int kCopies2 = 2, kCopiesB = 3, kCopiesHistB = 4, kCopiesS = 4;
constexpr int kCopiesA = 3, kCopiesHistA = 4;

// The iterations after layer l's own in which its stages run.
struct Lags {
  int p1, p2, pool, list, pick, cal, score, cand, fin;
};
// wide: pass 1, pass 2 and the select stages share a launch (small grids), else
// the K passes of a layer run before the select launch of its iteration.
constexpr Lags stage_lags(bool wide, bool given_lse, bool adaptive) {
  const int p2 = wide && !given_lse ? 1 : 0;
  const int cal = p2 + (wide ? 1 : 0) + (adaptive ? kAllocLag : 0);
  return Lags{0, p2, cal - 3, cal - 2, cal - 1, cal, cal + 1, cal + 2, cal + 3};
}
constexpr int kLongestLag = stage_lags(true, false, true).fin;
constexpr int kCopiesTab = kLongestLag + 1;

// Copies of B and of its histogram: without the wide passes no launch lies
// between pass 2 and the calibration, so one fewer is enough.
constexpr int copies_b(bool wide, bool adaptive) { return kCopiesB - !wide + (adaptive ? kAllocLag : 0); }
constexpr int copies_hist_b(bool wide, bool adaptive) { return kCopiesHistB - !wide + (adaptive ? kAllocLag : 0); }
// Slots of the E history (layer l writes slot l mod their number): the m that a
// persistence term reads, the layer's own and one per layer whose pass 2 runs
// before or beside the calibration that reads them.
constexpr int history_slots(int m, bool adaptive) { return m + 2 + (adaptive ? kAllocLag : 0); }

}  // namespace bacon
