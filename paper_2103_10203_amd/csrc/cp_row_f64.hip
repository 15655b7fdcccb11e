// Component-parallel row kernels, 2D, FP64 (Hooke phases); the dispatch over
// all row families.
#include "cp_rb.h"
#include "solve_cp.h"

using namespace mor_cp;

namespace {
template <int NH, int MODE>
bool go(int rows, const CpArgs& a) {
  using F = RowF<3, NH, MAT_HOOKE>;
  constexpr int RB = row_rb(3, NH / F::RL, NH, true, false);
  const dim3 g((rows + RB - 1) / RB, (unsigned)a.nrve);
  k_row_cp<double, MatDev64, 3, NH, RB, MODE, MAT_HOOKE>
      <<<g, whole_waves(3 * RB * (NH / F::RL)), row_cp_lds<NH, RB, 3, double>(), a.st>>>(
          a.plans, a.list, a.state, (cpx<double>*)a.yl, a.off, *a.mat64, nullptr, a.eps, a.sig, a.sigpart, a.dec);
  return true;
}
template <int NH>
bool length(int mode, int rows, const CpArgs& a) {
  return mode == CP_ITER ? go<NH, MODE_ITER>(rows, a) : go<NH, MODE_FINAL>(rows, a);
}

template <int C, int NH>
int rb_of(bool fp64, bool j2) {
  if (j2) return row_rb(C, NH / RowF<C, NH, MAT_J2>::RL, NH, fp64, true);
  return row_rb(C, NH / RowF<C, NH, MAT_HOOKE>::RL, NH, fp64, false);
}
}  // namespace

bool cp_row_2d_f64(int nh, int mode, int rows, const CpArgs& a) {
  switch (nh) {
    case 16: return length<16>(mode, rows, a);
    case 18: return length<18>(mode, rows, a);
    case 24: return length<24>(mode, rows, a);
    case 27: return length<27>(mode, rows, a);
    case 32: return length<32>(mode, rows, a);
    case 36: return length<36>(mode, rows, a);
    case 48: return length<48>(mode, rows, a);
    case 54: return length<54>(mode, rows, a);
    case 64: return length<64>(mode, rows, a);
    case 72: return length<72>(mode, rows, a);
    case 81: return length<81>(mode, rows, a);
    case 96: return length<96>(mode, rows, a);
    case 108: return length<108>(mode, rows, a);
    case 128: return length<128>(mode, rows, a);
    case 144: return length<144>(mode, rows, a);
    case 162: return length<162>(mode, rows, a);
    case 192: return length<192>(mode, rows, a);
    case 216: return length<216>(mode, rows, a);
    case 256: return length<256>(mode, rows, a);
    default: return false;
  }
}

int cp_row_rb(int C, int nh, bool fp64, bool j2) {
  if (C == 6 && fp64) return 0;
  if (!row_new(C, nh) && !row_shared(C, nh)) return 0;
#define MOR_RB(N)                                             \
  case N: return C == 3 ? rb_of<3, N>(fp64, j2) : rb_of<6, N>(fp64, j2);
  switch (nh) {
    MOR_RB(12) MOR_RB(16) MOR_RB(18) MOR_RB(24) MOR_RB(27) MOR_RB(32) MOR_RB(36) MOR_RB(48) MOR_RB(54) MOR_RB(64)
    MOR_RB(72) MOR_RB(81) MOR_RB(96) MOR_RB(108) MOR_RB(128) MOR_RB(144) MOR_RB(162) MOR_RB(192) MOR_RB(216)
    MOR_RB(256)
    default: return 0;
  }
#undef MOR_RB
}

bool cp_row_only(int C, int nh, bool fp64) {
  return fp64 ? C == 3 && (row_new(3, nh) || row_shared(3, nh)) : row_new(C, nh);
}

bool cp_row(int C, int nh, bool fp64, bool j2, int mode, int rows, const CpArgs& a) {
  if (fp64) return C == 3 && !j2 && cp_row_2d_f64(nh, mode, rows, a);
  return C == 3 ? cp_row_2d(nh, j2, mode, rows, a) : cp_row_3d(nh, j2, mode, rows, a);
}
