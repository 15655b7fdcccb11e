// Column kernels of the lengths outside ColCfg, FP32 and FP64.
#include "solve_cp.h"

using namespace mor_cp;

namespace {
template <typename T, typename MT, int C, int N0, int MODE>
void go(int ncol, const CpArgs& a, const MT& mat) {
  using Cfg = ColAny<C, N0>;
  const dim3 g((ncol + Cfg::CB - 1) / Cfg::CB, (unsigned)a.nrve);
  k_col_any<T, MT, C, N0, MODE><<<g, col_nt<C, N0, Cfg>(), col_lds<C, N0, Cfg, T>(), a.st>>>(
      a.plans, a.list, a.state, a.ebar, (cpx<T>*)a.yc, (cpx<T>*)a.coef, a.warm, a.off, a.part, mat);
}

constexpr bool col_new(int C, int n0) {
  return n0 == 24 || n0 == 32 || n0 == 36 || n0 == 48 || n0 == 54 || n0 == 72 || n0 == 96 || n0 == 108 ||
         (C == 3 && (n0 == 144 || n0 == 162 || n0 == 192 || n0 == 216 || n0 == 288 || n0 == 324 || n0 == 432));
}
constexpr bool col_f64(int C, int n0) {
  return C == 3 && n0 != 24 && (col_new(3, n0) || n0 == 64 || n0 == 128 || n0 == 256 || n0 == 384 || n0 == 512);
}

template <int C, int N0>
bool length(bool fp64, int mode, int ncol, const CpArgs& a) {
  if (fp64) {
    if constexpr (col_f64(C, N0)) {
      if (mode == CP_ITER) go<double, MatDev64, C, N0, MODE_ITER>(ncol, a, *a.mat64);
      else go<double, MatDev64, C, N0, MODE_INIT>(ncol, a, *a.mat64);
      return true;
    }
  } else {
    if constexpr (col_new(C, N0)) {
      if (mode == CP_ITER) go<float, MatDev, C, N0, MODE_ITER>(ncol, a, *a.mat);
      else go<float, MatDev, C, N0, MODE_INIT>(ncol, a, *a.mat);
      return true;
    }
  }
  return false;
}
}  // namespace

#define MOR_COLS(X) \
  X(24) X(32) X(36) X(48) X(54) X(64) X(72) X(96) X(108) X(128) X(144) X(162) X(192) X(216) X(256) X(288) X(324) X(384) \
  X(432) X(512)

int cp_col_cb(int C, int n0, bool fp64) {
  if (fp64 ? !col_f64(C, n0) : !col_new(C, n0)) return 0;
#define X(N) case N: return C == 3 ? ColAny<3, N>::CB : ColAny<6, N>::CB;
  switch (n0) { MOR_COLS(X) default: return 0; }
#undef X
}

bool cp_col(int C, int n0, bool fp64, int mode, int ncol, const CpArgs& a) {
#define X(N) case N: return C == 3 ? length<3, N>(fp64, mode, ncol, a) : length<6, N>(fp64, mode, ncol, a);
  switch (n0) { MOR_COLS(X) default: return false; }
#undef X
}
