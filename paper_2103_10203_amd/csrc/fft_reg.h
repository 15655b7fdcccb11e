// Compile-time specialised FFT building blocks: length-R DFTs in registers
// and in-place Stockham passes over an LDS buffer.
//
// Stockham pass (radix R, span P = product of the radices before it, length
// N): butterfly i < N/R of a sequence reads x[i + j N/R] (j < R), multiplies
// input j by w^{j k N/(P R)} with k = i mod P and w = exp(SIGN 2 pi i / N),
// applies the length-R DFT and stores output j at (i - k) R + k + j P.  A
// pass reads everything into registers, waits at a barrier, then writes in
// place, so one LDS buffer suffices.  The last pass of a transform leaves
// thread i holding outputs i + j N/R; the first pass (P = 1) of the next
// transform with the same radix reads exactly those indices, so pointwise
// work between an inverse and a forward transform needs no LDS round trip.
#pragma once

#include "fft_lds.h"

namespace fftr {

template <int SIGN, typename T>
__device__ __forceinline__ cpx<T> mul_i(cpx<T> a) {
  return SIGN > 0 ? cpx<T>{-a.y, a.x} : cpx<T>{a.y, -a.x};
}

// cos and sin of 2 pi k / 16 for k = 0..8
__host__ __device__ constexpr double c16(int k) {
  return k == 0 ? 1.0 : k == 1 ? 0.92387953251128674 : k == 2 ? 0.70710678118654752
       : k == 3 ? 0.38268343236508977 : k == 4 ? 0.0 : k == 5 ? -0.38268343236508977
       : k == 6 ? -0.70710678118654752 : k == 7 ? -0.92387953251128674 : -1.0;
}
__host__ __device__ constexpr double s16(int k) {
  return k == 0 ? 0.0 : k == 1 ? 0.38268343236508977 : k == 2 ? 0.70710678118654752
       : k == 3 ? 0.92387953251128674 : k == 4 ? 1.0 : k == 5 ? 0.92387953251128674
       : k == 6 ? 0.70710678118654752 : k == 7 ? 0.38268343236508977 : 0.0;
}

template <int SIGN, int K, typename T>
__device__ __forceinline__ cpx<T> rot16(cpx<T> a) {
  // a * exp(SIGN 2 pi i K / 16), K in [0, 8)
  if constexpr (K == 0) return a;
  else if constexpr (K == 4) return mul_i<SIGN>(a);
  else {
    constexpr T c = (T)c16(K);
    constexpr T s = (T)(SIGN * s16(K));
    return cmul_mad(a, cpx<T>{c, s});
  }
}

template <int R, int SIGN>
struct Dft;

template <int SIGN>
struct Dft<2, SIGN> {
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <int SIGN>
struct Dft<3, SIGN> {
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    const T h = (T)0.86602540378443864676;
    cpx<T> u0 = v[0], u1 = v[1], u2 = v[2];
    cpx<T> sm = cadd(u1, u2);
    const cpx<T> d = mul_i<SIGN>(csub(u1, u2));
    const cpx<T> base = {mad(T(-0.5), sm.x, u0.x), mad(T(-0.5), sm.y, u0.y)};
    v[0] = cadd(u0, sm);
    v[1] = {mad(d.x, h, base.x), mad(d.y, h, base.y)};
    v[2] = {mad(d.x, -h, base.x), mad(d.y, -h, base.y)};
  }
};

template <int SIGN>
struct Dft<4, SIGN> {
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    cpx<T> s13 = cadd(v[1], v[3]), d13 = mul_i<SIGN>(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[1] = cadd(d02, d13);
    v[2] = csub(s02, s13);
    v[3] = csub(d02, d13);
  }
};

template <int SIGN>
struct Dft<6, SIGN> {
  // two length-3 DFTs of the even and odd samples, combined with w6^k
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> e[3] = {v[0], v[2], v[4]};
    cpx<T> o[3] = {v[1], v[3], v[5]};
    Dft<3, SIGN>::run(e);
    Dft<3, SIGN>::run(o);
    const T h = (T)0.86602540378443864676;
    // w6^1 = 1/2 + SIGN i h, w6^2 = -1/2 + SIGN i h
    const T hs = SIGN > 0 ? h : -h;
    const cpx<T> o1 = {mad(T(0.5), o[1].x, -mul_rn(hs, o[1].y)), mad(T(0.5), o[1].y, mul_rn(hs, o[1].x))};
    const cpx<T> o2 = {mad(T(-0.5), o[2].x, -mul_rn(hs, o[2].y)), mad(T(-0.5), o[2].y, mul_rn(hs, o[2].x))};
    v[0] = cadd(e[0], o[0]);
    v[3] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[4] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[5] = csub(e[2], o2);
  }
};

template <int SIGN>
struct Dft<8, SIGN> {
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> e[4] = {v[0], v[2], v[4], v[6]};
    cpx<T> o[4] = {v[1], v[3], v[5], v[7]};
    Dft<4, SIGN>::run(e);
    Dft<4, SIGN>::run(o);
    o[1] = rot16<SIGN, 2>(o[1]);
    o[2] = rot16<SIGN, 4>(o[2]);
    o[3] = rot16<SIGN, 6>(o[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 4] = csub(e[k], o[k]);
    }
  }
};

template <int SIGN>
struct Dft<9, SIGN> {
  // 3 x 3: length-3 DFTs over n1 of x[3 n1 + n2], twiddles w9^{n2 k1}, then
  // length-3 DFTs over n2; output k1 + 3 k2.
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    // cos and sin of 2 pi k / 9, k = 1, 2, 4
    const T c1 = (T)0.76604444311897803520, s1 = (T)(SIGN * 0.64278760968653932632);
    const T c2 = (T)0.17364817766693034885, s2 = (T)(SIGN * 0.98480775301220805937);
    const T c4 = (T)-0.93969262078590838405, s4 = (T)(SIGN * 0.34202014332566873304);
    cpx<T> a[3][3];
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[3 * n1 + n2];
      Dft<3, SIGN>::run(a[n2]);
    }
    a[1][1] = cmul_mad(a[1][1], {c1, s1});
    a[1][2] = cmul_mad(a[1][2], {c2, s2});
    a[2][1] = cmul_mad(a[2][1], {c2, s2});
    a[2][2] = cmul_mad(a[2][2], {c4, s4});
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      cpx<T> b[3] = {a[0][k1], a[1][k1], a[2][k1]};
      Dft<3, SIGN>::run(b);
#pragma unroll
      for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = b[k2];
    }
  }
};

template <int SIGN>
struct Dft<12, SIGN> {
  // Good-Thomas 3 x 4 (coprime factors, so no twiddles between the stages):
  // length-3 DFTs over n1 of x[(4 n1 + 3 n2) mod 12] for each n2, then
  // length-4 DFTs over n2 for each k1, output k = (4 k1 + 9 k2) mod 12.
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> a[4][3];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[(4 * n1 + 3 * n2) % 12];
      Dft<3, SIGN>::run(a[n2]);
    }
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      cpx<T> b[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
      Dft<4, SIGN>::run(b);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) v[(4 * k1 + 9 * k2) % 12] = b[k2];
    }
  }
};

template <int SIGN>
struct Dft<16, SIGN> {
  // 4 x 4: length-4 DFTs over n1 of x[4 n1 + n2], twiddles w16^{n2 k1}, then
  // length-4 DFTs over n2; output k1 + 4 k2.  Fewer operations than halving
  // into two length-8 DFTs (two of the nine twiddles are -i or its multiples
  // of pi/4 and no combining stage of 16 complex additions).
  template <typename T>
  __device__ __forceinline__ static void run(cpx<T>* v) {
    cpx<T> a[4][4];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
      a[n2][0] = v[n2];
      a[n2][1] = v[4 + n2];
      a[n2][2] = v[8 + n2];
      a[n2][3] = v[12 + n2];
      Dft<4, SIGN>::run(a[n2]);
    }
    a[1][1] = rot16<SIGN, 1>(a[1][1]);
    a[1][2] = rot16<SIGN, 2>(a[1][2]);
    a[1][3] = rot16<SIGN, 3>(a[1][3]);
    a[2][1] = rot16<SIGN, 2>(a[2][1]);
    a[2][2] = rot16<SIGN, 4>(a[2][2]);
    a[2][3] = rot16<SIGN, 6>(a[2][3]);
    a[3][1] = rot16<SIGN, 3>(a[3][1]);
    a[3][2] = rot16<SIGN, 6>(a[3][2]);
    a[3][3] = rot16<SIGN, 1>(a[3][3]);  // w16^9 = -w16^1: sign folded below
    a[3][3] = {-a[3][3].x, -a[3][3].y};
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      cpx<T> b[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
      Dft<4, SIGN>::run(b);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = b[k2];
    }
  }
};

// LDS position of element i of a sequence: one pad slot after every 16
// elements, so that stride-R accesses (R = 2..16, 8-byte elements) of a
// wavefront spread over all banks.
__host__ __device__ constexpr int pad16(int i) { return i + (i >> 4); }

// Data layout with one pad slot after every 2^PS elements (PS = 4: pad16).
template <int PS>
__host__ __device__ constexpr int padp(int i) {
  return i + (i >> PS);
}

// Sequence stride in LDS for `len` logical elements (odd, so that sequences
// start on different banks).
__host__ __device__ constexpr int seq_stride(int len) {
  return (pad16(len - 1) + 1) | 1;
}

// Twiddle w^{e} from a padded LDS table tw[pad16(t)] = exp(-2 pi i t / (N * TWS)),
// read at stride TWS (conjugated for SIGN > 0).
template <int SIGN, int TWS, typename T>
__device__ __forceinline__ cpx<T> twid(const cpx<T>* tw, int e) {
  cpx<T> w = tw[pad16(e * TWS)];  // tables are stored padded, like the data
  return SIGN > 0 ? cconj(w) : w;
}

// Apply the pass twiddles to v[1..R-1] for butterfly phase k.
template <int N, int R, int P, int SIGN, int TWS = 1, typename T>
__device__ __forceinline__ void pass_twiddle(cpx<T>* v, int k, const cpx<T>* tw) {
  if constexpr (P > 1) {
    constexpr int ST = N / (P * R);
#pragma unroll
    for (int j = 1; j < R; ++j) v[j] = cmul_mad(v[j], twid<SIGN, TWS>(tw, j * k * ST));
  }
}

// One in-place Stockham pass over NS sequences (base + s*SS, positions
// padded by padp<PS>) by NT threads.  TW = false skips the pass twiddles (the
// producer of the pass's input has applied them).  Work item t is butterfly
// i = t % NB of sequence s = t / NB, or with SF (sequence fastest) butterfly
// t / NS of sequence t % NS: neighbouring lanes then take the same butterfly
// of neighbouring sequences, which an odd sequence stride spreads over all
// banks where the butterflies of one sequence would collide.
template <int N, int R, int P, int SIGN, int NS, int SS, int NT, int TWS, int PS = 4, bool TW = true, bool SF = false,
          typename T>
__device__ __forceinline__ void lds_pass(cpx<T>* buf, const cpx<T>* tw, int tid) {
  constexpr int NB = N / R;
  constexpr int TOTAL = NS * NB;
  constexpr int PER = (TOTAL + NT - 1) / NT;
  cpx<T> v[PER][R];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int t = tid + q * NT;
    if (TOTAL % NT == 0 || t < TOTAL) {
      // (t / NS) % NB == t / NS here; the modulo tells the compiler i < NB
      const int s = SF ? t % NS : t / NB, i = SF ? (t / NS) % NB : t % NB;
      const int k = i % P;
      const cpx<T>* src = buf + s * SS;
#pragma unroll
      for (int j = 0; j < R; ++j) v[q][j] = src[padp<PS>(i + j * NB)];
      if constexpr (TW) pass_twiddle<N, R, P, SIGN, TWS>(v[q], k, tw);
      Dft<R, SIGN>::run(v[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int t = tid + q * NT;
    if (TOTAL % NT == 0 || t < TOTAL) {
      const int s = SF ? t % NS : t / NB, i = SF ? (t / NS) % NB : t % NB;
      const int k = i % P;
      cpx<T>* dst = buf + s * SS;
      const int o = (i - k) * R + k;
#pragma unroll
      for (int j = 0; j < R; ++j) dst[padp<PS>(o + j * P)] = v[q][j];
    }
  }
  __syncthreads();
}

template <int... Rs>
struct RList {};

// Runs the passes of RList in order starting with span P.
template <int N, int SIGN, int P, int NS, int SS, int NT, int TWS, int PS = 4, bool SF = false, typename T>
__device__ __forceinline__ void lds_passes(cpx<T>*, const cpx<T>*, int, RList<>) {}

template <int N, int SIGN, int P, int NS, int SS, int NT, int TWS, int PS = 4, bool SF = false, int R, int... Rest,
          typename T>
__device__ __forceinline__ void lds_passes(cpx<T>* buf, const cpx<T>* tw, int tid, RList<R, Rest...>) {
  lds_pass<N, R, P, SIGN, NS, SS, NT, TWS, PS, true, SF>(buf, tw, tid);
  lds_passes<N, SIGN, P * R, NS, SS, NT, TWS, PS, SF>(buf, tw, tid, RList<Rest...>{});
}

// Single radix of a one-element list (0 otherwise).
template <typename A>
struct Single {
  static constexpr int v = 0;
};
template <int R>
struct Single<RList<R>> {
  static constexpr int v = R;
};

template <int... Rs>
struct Prod;
template <>
struct Prod<> {
  static constexpr int v = 1;
};
template <int R, int... Rest>
struct Prod<R, Rest...> {
  static constexpr int v = R * Prod<Rest...>::v;
};

// Reverse of a radix list.
template <typename A, typename B>
struct Rev;
template <int... Bs>
struct Rev<RList<>, RList<Bs...>> {
  using type = RList<Bs...>;
};
template <int A0, int... As, int... Bs>
struct Rev<RList<A0, As...>, RList<Bs...>> {
  using type = typename Rev<RList<As...>, RList<A0, Bs...>>::type;
};

}  // namespace fftr
