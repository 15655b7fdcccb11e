// Host rules of a solve's schedule, without HIP, so that a CPU test compiles them.
#pragma once

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

}  // namespace mor_sched
