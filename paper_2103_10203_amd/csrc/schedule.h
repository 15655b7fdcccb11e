// Host rules of a solve's schedule, without HIP, so that a CPU test compiles them.
#pragma once

#include <algorithm>
#include <cstdint>

namespace mor_sched {

// Most workgroups (of four rows) for which the iteration rows of a row_fast
// length run on the component-parallel kernel instead.  It has a third of the
// chain per wavefront and four times the workgroups, but more LDS traffic per
// row, so it wins while the device has room: row_fast / component-parallel per
// solve, 256^2 with 1, 4, 8, 16 RVEs (64, 256, 512, 1024 workgroups) 753 / 637,
// 770 / 682, 801 / 785, 888 / 969 us; 384^2 with 1, 4 (96, 384) 889 / 699,
// 960 / 887; J2 paths of 512^2 with 1, 4 (128, 512) 9.3 / 7.9, 13.6 / 13.0 ms, of
// 128^2 with 16 (512) 7.3 / 5.8 ms; 64^2 with 16, 64, 256 (256, 1024, 4096)
// 484 / 421, 498 / 464, 587 / 704 us.
constexpr int64_t kCpFewMax = 512;

// One grid of a call, as far as the choice of its row kernel goes.
struct RowCall {
  bool row_fast;         // the length has a row_fast kernel
  bool default_variant;  // and its default variant is selected
  bool dft;              // the last axis is transformed by the partial DFT
  bool persistent;       // MOR_SCHED_PERSISTENT
  int64_t line_bytes;    // transform lines of the largest RVE
  int rb;                // rows per workgroup of the component-parallel kernel, 0: not built
  int64_t rows, rves;    // rows of an RVE, RVEs in the call
};

// Whether the iteration's rows run on the component-parallel kernel instead of
// row_fast: it has the factors and the bits of the default variant, 32-bit
// offsets, and a grid of its own only (the persistent schedule's queue is walked
// by row_fast).
inline bool rows_by_component(const RowCall& c) {
  if (!c.row_fast || !c.default_variant || c.dft || c.persistent) return false;
  if (c.line_bytes >= (int64_t(1) << 31) || c.rb == 0) return false;
  return (c.rows + c.rb - 1) / c.rb * c.rves <= kCpFewMax;
}

// Sub-batches: a grid's RVEs are cut into runs whose transform lines stay in the
// device's last-level cache, and the chunk of iterations of one run comes before
// that of the next.  Defaults: MI355X's 256 MB Infinity Cache less room for the
// coefficients, tables and phase maps the passes also stream; and no fewer RVEs
// than pay for the launches of a further run.
constexpr int64_t kRunBytes = (int64_t)192 << 20;
constexpr int64_t kRunRves = 128;

// Lanes: runs have nothing to do with each other, so some execute their chunks
// on streams of their own, forked from and joined to the solve's stream around
// every chunk.
//  * Several grids: a grid whose launches do not fill the device leaves CUs
//    idle, so grids run side by side, while the transform lines of all of them
//    fit the 256 MB Infinity Cache (beyond that they drive each other out), or
//    the run limit where the caller has lowered it: in turn / side by side, 16
//    RVEs each of 96x144, 162x108, 288x192 (12 MB) 1976 / 1168 us, of 128^2, 256^2,
//    384^2 64 each (80 MB) 4.36 / 3.32 ms, 512 each (630 MB) 24.2 / 24.7 ms.
//  * Otherwise two at a time, each within half the limit, so that one's row pass
//    (bound by VALU issue) overlaps the other's column pass (bound by latency), if
//    each has at least kPairWgs row workgroups and kPairBytes of lines; one at a
//    time / in pairs, inputs changing from call to call: 1024 RVEs of 256^2 12.70 /
//    12.43 ms, 512 each of 128^2, 256^2, 384^2 23.9 / 22.4, eight of 128^3 8.99 /
//    8.82, 16 of them 17.7 / 15.9, 192 of 256^2 2.70 / 2.49, 512 of 128^2 2.01 / 1.71,
//    1024 of 64^2 (10 MB each) 1.13 / 1.03; at the line no gain: 128 of 256^2 (1024
//    workgroups, 22 MB each) 1.84 / 1.84, 64 of 384^2 2.47 / 2.47; below it (one set
//    of inputs) 64 of 256^2 (512) 1.32 / 1.31, four of 48x72x96 (864) 1.69 / 1.76, 512
//    of 64^2 (1024, but 5 MB each) 0.73 / 0.77 ms.
constexpr int kLanes = 4;  // streams, the solve's own among them
constexpr int64_t kLanesBytes = (int64_t)256 << 20;
constexpr int64_t kPairWgs = 1024;
constexpr int64_t kPairBytes = (int64_t)6 << 20;

// Whether the grids of a call run side by side; bytes: the lines of all.
inline bool grids_side_by_side(int64_t grids, int64_t bytes, int64_t limit) {
  return grids > 1 && bytes <= (limit > 0 && limit < kRunBytes ? limit : kLanesBytes);
}

// A run that may share the device with another: within half the limit.
inline bool shares_device(int64_t run_bytes, int64_t limit) { return run_bytes <= limit / 2; }

struct Cut {
  int64_t runs;
  bool pairs;  // two at a time
};

// Runs of one grid of a call: the fewest within the limit, or, where pairs of
// runs are possible in the call and pay, the fewest even number of them within
// half of it.  A minimum of RVEs that the caller has set bounds every run; the
// default one bounds the runs that go one at a time, and workgroups and lines
// those in pairs (eight RVEs of 128^3 go as four runs).
inline Cut cut_runs(int64_t bytes, int64_t rves, int64_t row_wgs, int64_t limit, int64_t min_rves, bool pairs) {
  if (limit <= 0) return {1, false};
  auto ceil_div = [](int64_t a, int64_t b) { return a / b + (a % b != 0); };
  min_rves = std::max<int64_t>(1, min_rves);
  const int64_t one = std::max<int64_t>(1, std::min(ceil_div(bytes, limit), rves / min_rves));
  const int64_t two = std::max<int64_t>(2, (ceil_div(2 * bytes, limit) + 1) / 2 * 2);
  const int64_t least = min_rves == kRunRves ? 1 : min_rves;
  if (pairs && row_wgs / two >= kPairWgs && bytes / two >= kPairBytes && rves / two >= least) return {two, true};
  return {one, false};
}

}  // namespace mor_sched
