// Rows per workgroup of the component-parallel row kernel.
#pragma once

namespace mor_cp {

// Lengths row_fast has no kernel for.
constexpr bool row_new(int C, int nh) {
  return C == 3 ? (nh == 16 || nh == 18 || nh == 24 || nh == 27 || nh == 36 || nh == 48 || nh == 54 || nh == 72 ||
                   nh == 81 || nh == 96 || nh == 108 || nh == 144 || nh == 162 || nh == 216)
                : (nh == 12 || nh == 16 || nh == 18 || nh == 24 || nh == 27 || nh == 36 || nh == 48 || nh == 54);
}
// Lengths row_fast serves (default factors shared).
constexpr bool row_shared(int C, int nh) {
  return nh == 32 || nh == 64 || nh == 128 || (C == 3 && (nh == 192 || nh == 256));
}

// tr = threads per row and component.  Eight rows, so that a gathered run is
// 64 bytes (128 in FP64): with four, 288x192 takes 1.04-1.08 times as long from
// 4 RVEs on and 48x72x96 1.07, and gains 3 % for one RVE.  Sixteen where eight
// leave more than a fifth of the wavefronts empty; four where eight take more
// than 640 threads or leave room for fewer than three workgroups on a CU, with
// J2 phases (the plastic state, contiguous along the row, is most of the
// traffic) and on the shared lengths, where the kernel is the form for few
// workgroups.
constexpr int row_rb(int C, int tr, int nh, bool fp64, bool j2) {
  if (j2 || (!fp64 && row_shared(C, nh))) return 4;
  const int lds8 = C * 8 * (nh + nh / 16 + 3) * (fp64 ? 16 : 8);
  if (C * 8 * tr > 640 || lds8 > 48 * 1024) return 4;
  const int w = (C * 8 * tr + 63) / 64 * 64;
  if (!fp64 && 5 * C * 8 * tr < 4 * w && C * 16 * tr <= 640) return 16;
  return 8;
}

}  // namespace mor_cp
