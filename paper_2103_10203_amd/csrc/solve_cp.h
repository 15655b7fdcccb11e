// Component-parallel row kernel, and the column kernels of the lengths that
// solve_fast.h does not build: compile-time transforms in FP32 and FP64,
// launched through the plain functions at the end (each family is compiled in a
// source file of its own).  Built are, of the even 2^a 3^b lengths,
//   2D rows and columns  32 to 512 but 486, FP32 and FP64 (FP32 columns of 24 too)
//   3D rows              24 to 128, and 256, FP32
//   3D axes 0 and 1      24 to 128, FP32 (axis 1 in solve_fast.h)
// Every other length, and FP64 in 3D, runs the runtime-radix kernels of
// solve_kernels.h at about a third of the speed.
//
// The row kernel of solve_fast.h keeps all strain components of a thread's
// points in registers and transforms them one after the other: least LDS
// traffic, but a serial chain of C forward and C inverse transforms and 16
// rows per workgroup, so one RVE of 256^2 runs 16 workgroups of four waves
// that take 9 us each.  Here every component of a row has its own threads: the
// chain is one inverse and one forward transform, and the components meet in
// LDS for the constitutive law.
#pragma once

#include "solve_fast.h"

namespace mor_cp {

using namespace mor_k;

// Factorisation of a row of length 2 NH: register pass radix RL, inverse LDS
// passes RA (forward: reversed).  Lengths that row_fast also serves have the
// factors of its default.
template <int C, int NH, int MAT>
struct RowF;
template <int C, int MAT> struct RowF<C, 12, MAT>  { static constexpr int RL = 3; using RA = RList<4>; };
template <int C, int MAT> struct RowF<C, 16, MAT>  { static constexpr int RL = 4; using RA = RList<4>; };
template <int C, int MAT> struct RowF<C, 18, MAT>  { static constexpr int RL = 3; using RA = RList<6>; };
template <int C, int MAT> struct RowF<C, 24, MAT>  { static constexpr int RL = 4; using RA = RList<6>; };
template <int C, int MAT> struct RowF<C, 27, MAT>  { static constexpr int RL = 3; using RA = RList<9>; };
template <int C, int MAT> struct RowF<C, 32, MAT>  { static constexpr int RL = 4; using RA = RList<8>; };
template <int C, int MAT> struct RowF<C, 36, MAT>  { static constexpr int RL = 6; using RA = RList<6>; };
template <int C, int MAT> struct RowF<C, 48, MAT>  { static constexpr int RL = 6; using RA = RList<8>; };
template <int C, int MAT> struct RowF<C, 54, MAT>  { static constexpr int RL = 6; using RA = RList<9>; };
template <int MAT> struct RowF<3, 64, MAT>         { static constexpr int RL = 8; using RA = RList<8>; };
template <int MAT> struct RowF<6, 64, MAT>         { static constexpr int RL = 4; using RA = RList<4, 4>; };
template <int C, int MAT> struct RowF<C, 72, MAT>  { static constexpr int RL = 8; using RA = RList<9>; };
template <int C, int MAT> struct RowF<C, 81, MAT>  { static constexpr int RL = 9; using RA = RList<9>; };
template <int C, int MAT> struct RowF<C, 96, MAT>  { static constexpr int RL = 8; using RA = RList<12>; };
template <int C, int MAT> struct RowF<C, 108, MAT> { static constexpr int RL = 9; using RA = RList<12>; };
template <int MAT> struct RowF<3, 128, MAT>        { static constexpr int RL = 8; using RA = RList<16>; };
template <int MAT> struct RowF<6, 128, MAT>        { static constexpr int RL = 4; using RA = RList<8, 4>; };
template <int C, int MAT> struct RowF<C, 144, MAT> { static constexpr int RL = 9; using RA = RList<16>; };
template <int C, int MAT> struct RowF<C, 162, MAT> { static constexpr int RL = 9; using RA = RList<6, 3>; };
template <int C> struct RowF<C, 192, MAT_HOOKE>    { static constexpr int RL = 12; using RA = RList<16>; };
template <int C> struct RowF<C, 192, MAT_J2>       { static constexpr int RL = 4; using RA = RList<4, 4, 3>; };
template <int C, int MAT> struct RowF<C, 216, MAT> { static constexpr int RL = 9; using RA = RList<8, 3>; };
template <int C> struct RowF<C, 256, MAT_HOOKE>    { static constexpr int RL = 16; using RA = RList<16>; };
template <int C> struct RowF<C, 256, MAT_J2>       { static constexpr int RL = 4; using RA = RList<8, 8>; };

template <int NH, int RB, int C, typename T>
constexpr size_t row_cp_lds() {
  return (size_t)(row_tw_len<NH>() + C * RB * row_ss<NH>()) * sizeof(cpx<T>);
}

// 8- or 16-byte raw buffer access (FP32 or FP64 complex); a load whose offset
// lies at or beyond the resource's size returns zero without an access.
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ cpx<T> buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off) {
  if constexpr (sizeof(T) == 4) {
    return load_or_zero(rs, byte_off);
  } else {
    const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)byte_off, 0, 0);
    return {__hiloint2double(v.y, v.x), __hiloint2double(v.w, v.z)};
  }
}
template <typename T>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off, cpx<T> a) {
  if constexpr (sizeof(T) == 4) {
    store_c(rs, byte_off, a);
  } else {
    const i32x4 v = {__double2loint(a.x), __double2hiint(a.x), __double2loint(a.y), __double2hiint(a.y)};
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)byte_off, 0, 0);
  }
}

// Workgroup = RB rows of one RVE, TR = NH / RL threads per row and component.
// Bound by the latency of its chain where few workgroups run, else by VALU
// issue.  Against the runtime-radix kernel it replaces on the lengths of
// row_new (two LDS buffers, integer division per butterfly): 16 RVEs each of
// 96x144, 162x108, 288x192 26.3 -> 10.4 us a launch (mean), four of 48x72x96
// 64 -> 23 us; FP64, 256 RVEs of 64^2 33.6 -> 14.4 us.
// MODE_ITER: Yl (F) -> Yl (T); MODE_FINAL: fields, stress sums, J2 state.
template <typename T, typename MT, int C, int NH, int RB, int MODE, int MAT>
__global__ __launch_bounds__(whole_waves(C * RB * (NH / RowF<C, NH, MAT>::RL))) void k_row_cp(
    const PlanDev* __restrict__ plans, const int* __restrict__ rve_list, RveState* __restrict__ st,
    cpx<T>* __restrict__ Yl, Offs off, MT mat, float* __restrict__ jstate, float* __restrict__ out_eps,
    float* __restrict__ out_sig, double* __restrict__ sig_part, Decide dec) {
  using F = RowF<C, NH, MAT>;
  constexpr int RL = F::RL, TR = NH / RL;
  constexpr int NSEQ = C * RB, NA = NSEQ * TR, NT = whole_waves(NA);
  constexpr int SS = row_ss<NH>();
  constexpr int S = Comp<C>::S, NST = Comp<C>::NST;
  constexpr int L = 2 * NH, KH = NH / 2 + 1;
  constexpr uint32_t ES = sizeof(cpx<T>);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ int lk[NH + 1];
  __shared__ uint32_t kofs[NH + 1];
  __shared__ int stopped;
  const int tid = threadIdx.x;
  __builtin_assume(tid >= 0 && tid < NT);
  const int b = rve_list[blockIdx.y], tile = blockIdx.x;
  if (MODE == MODE_ITER && !st[b].active) return;
  const PlanDev& P = plans[st[b].plan];
  const int rows = P.rows;
  const int r0 = tile * RB;
  if (r0 >= rows) return;
  const int nr = min(RB, rows - r0);
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem_raw);  // exp(-2 pi i t / L)
  cpx<T>* buf = tw + row_tw_len<NH>();               // sequence c * RB + row
  const int nlast = P.nlast;
  // stop decision of the previous iteration, as in row_tile
  const bool decide = MODE == MODE_ITER && dec.part != nullptr;
  const double* dpart = nullptr;
  int dnum = 0;
  double dp0 = 0.0, dp1 = 0.0;
  if (decide && tid < 64) {
    dpart = dec.part + off.part[b];
    dnum = (P.ncol + dec.cb - 1) / dec.cb;
    if (tid < dnum) dp0 = dpart[tid];
    if (tid + 64 < dnum) dp1 = dpart[tid + 64];
  }
  const cpx<T>* __restrict__ rtw_g = PT<T>::rtw(P);
  for (int t = tid; t < L; t += NT) tw[pad16(t)] = rtw_g[t];
  for (int t = tid; t <= NH; t += NT) kofs[t] = kOutOfRange;
  for (int t = tid; t < nlast; t += NT) lk[t] = P.last_k[t];
  __syncthreads();
  // all components span C * nlast * rows * ES < 2^31 bytes (checked by the host)
  for (int t = tid; t < nlast; t += NT) kofs[lk[t]] = (uint32_t)t * (uint32_t)rows * ES;
  __syncthreads();
  const uint32_t cbytes = (uint32_t)nlast * (uint32_t)rows * ES;  // one component
  const __amdgpu_buffer_rsrc_t rs =
      comp_rsrc(reinterpret_cast<const cpx<float>*>(Yl + off.yl[b]), (uint32_t)C * cbytes);

  // ---- gather of the half spectra, packed to length NH (see row_tile): item
  // (c, k, row), rows fastest; rows past the end read entries that are never
  // used or zero
  {
    constexpr int GT = C * KH * RB, GU = (GT + NT - 1) / NT;
    cpx<T> xa[GU], xb[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const int t = tid + u * NT;
      if (GT % NT == 0 || t < GT) {
        const int r = t % RB, k = (t / RB) % KH, c = t / (RB * KH);
        const uint32_t o = (uint32_t)c * cbytes + (uint32_t)(r0 + r) * ES;
        xa[u] = buf_load<T>(rs, kofs[k] + o);
        xb[u] = buf_load<T>(rs, kofs[NH - k] + o);
      }
    }
    if (decide && tid < 64) {
      const double sum = part_sum(dpart, dnum, tid, dp0, dp1);
      if (tid == 0) {
        double res = 0.0;
        const int end = stop_rule(st[b], sum, &res);
        stopped = end >= 0;
        if (tile == 0) stop_rve(st[b], end, res, dec.active);
      }
    }
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const int t = tid + u * NT;
      if (GT % NT == 0 || t < GT) {
        const int r = t % RB, k = (t / RB) % KH, c = t / (RB * KH);
        cpx<T>* x = buf + (c * RB + r) * SS;
        const cpx<T> a = cadd(xa[u], cconj(xb[u]));
        const cpx<T> d = cmul_mad(csub(xa[u], cconj(xb[u])), cconj(tw[pad16(k)]));
        x[pad16(k)] = {a.x - d.y, a.y + d.x};
        if (k != 0 && 2 * k != NH) x[pad16(NH - k)] = {a.x + d.y, d.x - a.y};
      }
    }
  }
  __syncthreads();
  if (decide && stopped) return;

  // ---- inverse: LDS passes, then the register pass back to the positions
  // the thread has read
  fftr::lds_passes<NH, +1, 1, NSEQ, SS, NT, 2, 4, true>(buf, tw, tid, typename F::RA{});
  const int s = tid / TR, i = tid % TR;
  const bool seq_live = NA == NT || s < NSEQ;
  cpx<T>* seq = buf + s * SS;
  cpx<T> v[RL], rtw[RL];
  if (seq_live) {
#pragma unroll
    for (int j = 0; j < RL; ++j) rtw[j] = fftr::twid<+1, 2>(tw, j * i * (NH / (TR * RL)));
#pragma unroll
    for (int j = 0; j < RL; ++j) v[j] = seq[pad16(i + j * TR)];
#pragma unroll
    for (int j = 1; j < RL; ++j) v[j] = cmul_mad(v[j], rtw[j]);
    Dft<RL, +1>::run(v);
#pragma unroll
    for (int j = 0; j < RL; ++j) seq[pad16(i + j * TR)] = v[j];
  }
  __syncthreads();

  // ---- pointwise step a): item (row, pair of points), pairs fastest
  double acc[S];
#pragma unroll
  for (int q = 0; q < S; ++q) acc[q] = 0.0;
  constexpr int PT_ = RB * NH, PU = (PT_ + NT - 1) / NT;
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int t = tid + u * NT;
    const int r = t / NH, p = t % NH;
    if ((PT_ % NT == 0 || t < PT_) && r < nr) {
      const int64_t p0 = (int64_t)(r0 + r) * L + 2 * p;
      const uchar2 gg = *reinterpret_cast<const uchar2*>(P.g + p0);
      cpx<T>* x = buf + r * SS + pad16(p);
      T e0[C], e1[C], t0[C], t1[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const cpx<T> z = x[c * RB * SS];
        e0[c] = z.x;
        e1[c] = z.y;
      }
      float sin0[NST], sin1[NST];
      if (MAT == MAT_J2) {
        const float* sp = jstate + off.field[b] * NST;
#pragma unroll
        for (int q = 0; q < NST; ++q) {
          const float2 w = *reinterpret_cast<const float2*>(sp + (int64_t)q * P.N + p0);
          sin0[q] = w.x;
          sin1[q] = w.y;
        }
      }
      if (MODE == MODE_ITER) {
        law<C, MAT, T>(e0, gg.x, mat, sin0, t0, (T*)nullptr, nullptr);
        law<C, MAT, T>(e1, gg.y, mat, sin1, t1, (T*)nullptr, nullptr);
#pragma unroll
        for (int c = 0; c < C; ++c) x[c * RB * SS] = {t0[c], t1[c]};
      } else {
        T s0[S], s1[S];
        float so0[NST], so1[NST];
        law<C, MAT, T>(e0, gg.x, mat, sin0, t0, s0, so0);
        law<C, MAT, T>(e1, gg.y, mat, sin1, t1, s1, so1);
        if (MAT == MAT_J2) {
          float* sp = jstate + off.field[b] * NST;
#pragma unroll
          for (int q = 0; q < NST; ++q)
            *reinterpret_cast<float2*>(sp + (int64_t)q * P.N + p0) = make_float2(so0[q], so1[q]);
        }
        if (out_eps) {
          float* fe = out_eps + off.field[b] * C;
#pragma unroll
          for (int c = 0; c < C; ++c)
            *reinterpret_cast<float2*>(fe + (int64_t)c * P.N + p0) = make_float2((float)e0[c], (float)e1[c]);
        }
        if (out_sig) {
          float* fs = out_sig + off.field[b] * S;
#pragma unroll
          for (int q = 0; q < S; ++q)
            *reinterpret_cast<float2*>(fs + (int64_t)q * P.N + p0) = make_float2((float)s0[q], (float)s1[q]);
        }
#pragma unroll
        for (int q = 0; q < S; ++q) acc[q] += (double)s0[q] + (double)s1[q];
      }
    }
  }
  if (MODE == MODE_FINAL) {
    __shared__ double red[(NT / 64) * S];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
      for (int q = 0; q < S; ++q) acc[q] += __shfl_down(acc[q], o, 64);
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int q = 0; q < S; ++q) red[(tid >> 6) * S + q] = acc[q];
    }
    __syncthreads();
    if (tid < S) {
      double w = 0.0;
      for (int q = 0; q < NT / 64; ++q) w += red[q * S + tid];
      sig_part[(off.part[b] + tile) * S + tid] = w;
    }
    return;
  }
  __syncthreads();

  // ---- forward: register pass, LDS passes, unpack at the sampled frequencies
  constexpr int R2 = fftr::Single<typename F::RA>::v;
  constexpr bool kPreTwiddle = R2 * RL == NH;  // as in row_tile
  if (seq_live) {
#pragma unroll
    for (int j = 0; j < RL; ++j) v[j] = seq[pad16(i + j * TR)];
    Dft<RL, -1>::run(v);
    if constexpr (kPreTwiddle) {
#pragma unroll
      for (int j = 1; j < RL; ++j) v[j] = cmul_mad(v[j], cconj(rtw[j]));
    }
  }
  __syncthreads();
  if (seq_live) {
#pragma unroll
    for (int j = 0; j < RL; ++j) seq[pad16(i * RL + j)] = v[j];
  }
  __syncthreads();
  if constexpr (kPreTwiddle) {
    fftr::lds_pass<NH, R2, RL, -1, NSEQ, SS, NT, 2, 4, false, true>(buf, tw, tid);
  } else {
    fftr::lds_passes<NH, -1, RL, NSEQ, SS, NT, 2, 4, true>(buf, tw, tid,
                                                           typename fftr::Rev<typename F::RA, RList<>>::type{});
  }
  for (int t = tid; t < C * nlast * RB; t += NT) {
    const int r = t % RB, q = t / RB;
    if (r >= nr) continue;
    int c = 0, j = q;
#pragma unroll
    for (int h = 1; h < C; ++h) {  // q = c * nlast + j without a division
      const bool up = j >= nlast;
      c += up;
      j -= up ? nlast : 0;
    }
    const int k = lk[j];
    const cpx<T>* z = buf + (c * RB + r) * SS;
    const cpx<T> Zk = z[pad16(k == NH ? 0 : k)];
    const cpx<T> Zc = cconj(z[pad16(k == 0 ? 0 : NH - k)]);
    const cpx<T> sm = cadd(Zk, Zc);
    const cpx<T> wd = cmul_mad(tw[pad16(k)], csub(Zk, Zc));
    buf_store<T>(rs, (uint32_t)c * cbytes + (uint32_t)j * (uint32_t)rows * ES + (uint32_t)(r0 + r) * ES,
                 {T(0.5) * (sm.x + wd.y), T(0.5) * (sm.y - wd.x)});
  }
}

// Columns of the lengths ColCfg does not list (and of those it does, in
// FP64, with the factors of its default variants): register pass RF, LDS
// passes FA, and CB columns per workgroup so that C CB N0 / RF threads nearly
// fill three to four wavefronts.
template <int N0>
struct ColF;
template <> struct ColF<24>  { static constexpr int RF = 4;  using FA = RList<6>; };
template <> struct ColF<32>  { static constexpr int RF = 4;  using FA = RList<8>; };
template <> struct ColF<36>  { static constexpr int RF = 6;  using FA = RList<6>; };
template <> struct ColF<48>  { static constexpr int RF = 6;  using FA = RList<8>; };
template <> struct ColF<54>  { static constexpr int RF = 6;  using FA = RList<9>; };
template <> struct ColF<64>  { static constexpr int RF = 8;  using FA = RList<8>; };
template <> struct ColF<72>  { static constexpr int RF = 8;  using FA = RList<9>; };
template <> struct ColF<96>  { static constexpr int RF = 8;  using FA = RList<12>; };
template <> struct ColF<108> { static constexpr int RF = 9;  using FA = RList<12>; };
template <> struct ColF<128> { static constexpr int RF = 8;  using FA = RList<4, 4>; };
template <> struct ColF<144> { static constexpr int RF = 9;  using FA = RList<4, 4>; };
template <> struct ColF<162> { static constexpr int RF = 9;  using FA = RList<6, 3>; };
template <> struct ColF<192> { static constexpr int RF = 8;  using FA = RList<6, 4>; };
template <> struct ColF<216> { static constexpr int RF = 6;  using FA = RList<6, 6>; };
template <> struct ColF<256> { static constexpr int RF = 8;  using FA = RList<8, 4>; };
template <> struct ColF<288> { static constexpr int RF = 6;  using FA = RList<8, 6>; };
template <> struct ColF<324> { static constexpr int RF = 6;  using FA = RList<9, 6>; };
template <> struct ColF<384> { static constexpr int RF = 6;  using FA = RList<8, 8>; };
template <> struct ColF<432> { static constexpr int RF = 6;  using FA = RList<9, 8>; };
template <> struct ColF<512> { static constexpr int RF = 8;  using FA = RList<8, 8>; };

template <int C, int N0>
struct ColAny : ColF<N0> {
  static constexpr int CB = (C * (N0 / ColF<N0>::RF) >= 192) ? 1 : 192 / (C * (N0 / ColF<N0>::RF));
};

// Against the runtime-radix kernel: 16 RVEs each of 96x144, 162x108, 288x192
// 31.0 -> 8.2 us a launch (mean), four of 48x72x96 37 -> 8.6 us; FP64, 256 RVEs
// of 64^2 25.6 -> 10.7 us.
template <typename T, typename MT, int C, int N0, int MODE>
__global__ __launch_bounds__((col_nt<C, N0, ColAny<C, N0>>())) void k_col_any(
    const PlanDev* __restrict__ plans, const int* __restrict__ rve_list, RveState* __restrict__ st,
    const double* __restrict__ ebar, cpx<T>* __restrict__ Yc, cpx<T>* __restrict__ coef,
    const cpx<float>* __restrict__ warm, Offs off, double* __restrict__ part, MT mat) {
  col_tile<C, N0, ColAny<C, N0>, MODE, T, MT>(plans, rve_list[blockIdx.y], blockIdx.x, st, ebar, Yc, coef, warm, off,
                                              part, mat, threadIdx.x);
}

}  // namespace mor_cp

// ------------------------------------------------------------------ launches
// One launch over a group of RVEs of one grid.
struct CpArgs {
  hipStream_t st;
  const PlanDev* plans;
  const int* list;
  int nrve;
  RveState* state;
  void* yl;    // cpx<float> or cpx<double>, as coef and yc
  void* yc;
  void* coef;
  const double* ebar;
  const cpx<float>* warm;
  mor_k::Offs off;
  double* part;
  const MatDev* mat;
  const MatDev64* mat64;
  float* jstate;
  float* eps;
  float* sig;
  double* sigpart;
  mor_k::Decide dec;
};
enum { CP_ITER = 0, CP_FINAL = 1, CP_INIT = 1 };

// Rows per workgroup of the component-parallel row kernel for rows of length
// 2 nh (0: not built).
int cp_row_rb(int C, int nh, bool fp64, bool j2);
// Lengths whose row passes run on it in every case (row_fast has no kernel).
bool cp_row_only(int C, int nh, bool fp64);
// The launch; false if that form is not built.
bool cp_row(int C, int nh, bool fp64, bool j2, int mode, int rows, const CpArgs& a);
// Columns per workgroup (0: not built) and the launch.
int cp_col_cb(int C, int n0, bool fp64);
bool cp_col(int C, int n0, bool fp64, int mode, int ncol, const CpArgs& a);
// per-family parts of cp_row
bool cp_row_2d(int nh, bool j2, int mode, int rows, const CpArgs& a);
bool cp_row_2d_f64(int nh, int mode, int rows, const CpArgs& a);
bool cp_row_3d(int nh, bool j2, int mode, int rows, const CpArgs& a);
