// Component-parallel row kernels, 3D, FP32.
#include "cp_rb.h"
#include "solve_cp.h"

using namespace mor_cp;

namespace {
template <int NH, int MODE, int MAT>
bool go(int rows, const CpArgs& a) {
  constexpr int TR = NH / RowF<6, NH, MAT>::RL;
  constexpr int RB = row_rb(6, TR, NH, false, MAT == MAT_J2);
  const dim3 g((rows + RB - 1) / RB, (unsigned)a.nrve);
  k_row_cp<float, MatDev, 6, NH, RB, MODE, MAT>
      <<<g, whole_waves(6 * RB * TR), row_cp_lds<NH, RB, 6, float>(), a.st>>>(
          a.plans, a.list, a.state, (cpx<float>*)a.yl, a.off, *a.mat, a.jstate, a.eps, a.sig, a.sigpart, a.dec);
  return true;
}

template <int NH>
bool length(bool j2, int mode, int rows, const CpArgs& a) {
  if (mode == CP_ITER)
    return j2 ? go<NH, MODE_ITER, MAT_J2>(rows, a) : go<NH, MODE_ITER, MAT_HOOKE>(rows, a);
  if constexpr (row_new(6, NH))  // the shared lengths finish on row_fast
    return j2 ? go<NH, MODE_FINAL, MAT_J2>(rows, a) : go<NH, MODE_FINAL, MAT_HOOKE>(rows, a);
  return false;
}
}  // namespace

bool cp_row_3d(int nh, bool j2, int mode, int rows, const CpArgs& a) {
  switch (nh) {
    case 12: return length<12>(j2, mode, rows, a);
    case 16: return length<16>(j2, mode, rows, a);
    case 18: return length<18>(j2, mode, rows, a);
    case 24: return length<24>(j2, mode, rows, a);
    case 27: return length<27>(j2, mode, rows, a);
    case 32: return length<32>(j2, mode, rows, a);
    case 36: return length<36>(j2, mode, rows, a);
    case 48: return length<48>(j2, mode, rows, a);
    case 54: return length<54>(j2, mode, rows, a);
    case 64: return length<64>(j2, mode, rows, a);
    case 128: return length<128>(j2, mode, rows, a);
    default: return false;
  }
}
