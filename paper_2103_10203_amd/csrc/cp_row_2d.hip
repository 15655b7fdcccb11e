// Component-parallel row kernels, 2D, FP32.
#include "cp_rb.h"
#include "solve_cp.h"

using namespace mor_cp;

namespace {
template <int NH, int MODE, int MAT>
bool go(int rows, const CpArgs& a) {
  constexpr int TR = NH / RowF<3, NH, MAT>::RL;
  constexpr int RB = row_rb(3, TR, NH, false, MAT == MAT_J2);
  const dim3 g((rows + RB - 1) / RB, (unsigned)a.nrve);
  k_row_cp<float, MatDev, 3, NH, RB, MODE, MAT>
      <<<g, whole_waves(3 * RB * TR), row_cp_lds<NH, RB, 3, float>(), a.st>>>(
          a.plans, a.list, a.state, (cpx<float>*)a.yl, a.off, *a.mat, a.jstate, a.eps, a.sig, a.sigpart, a.dec);
  return true;
}

template <int NH>
bool length(bool j2, int mode, int rows, const CpArgs& a) {
  if (mode == CP_ITER)
    return j2 ? go<NH, MODE_ITER, MAT_J2>(rows, a) : go<NH, MODE_ITER, MAT_HOOKE>(rows, a);
  if constexpr (row_new(3, NH))  // the shared lengths finish on row_fast
    return j2 ? go<NH, MODE_FINAL, MAT_J2>(rows, a) : go<NH, MODE_FINAL, MAT_HOOKE>(rows, a);
  return false;
}
}  // namespace

bool cp_row_2d(int nh, bool j2, int mode, int rows, const CpArgs& a) {
  switch (nh) {
    case 16: return length<16>(j2, mode, rows, a);
    case 18: return length<18>(j2, mode, rows, a);
    case 24: return length<24>(j2, mode, rows, a);
    case 27: return length<27>(j2, mode, rows, a);
    case 32: return length<32>(j2, mode, rows, a);
    case 36: return length<36>(j2, mode, rows, a);
    case 48: return length<48>(j2, mode, rows, a);
    case 54: return length<54>(j2, mode, rows, a);
    case 64: return length<64>(j2, mode, rows, a);
    case 72: return length<72>(j2, mode, rows, a);
    case 81: return length<81>(j2, mode, rows, a);
    case 96: return length<96>(j2, mode, rows, a);
    case 108: return length<108>(j2, mode, rows, a);
    case 128: return length<128>(j2, mode, rows, a);
    case 144: return length<144>(j2, mode, rows, a);
    case 162: return length<162>(j2, mode, rows, a);
    case 192: return length<192>(j2, mode, rows, a);
    case 216: return length<216>(j2, mode, rows, a);
    case 256: return length<256>(j2, mode, rows, a);
    default: return false;
  }
}
