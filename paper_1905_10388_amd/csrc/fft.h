// Transforms of B sequences of a length M known at compile time by one block,
// from registers to registers: every stage's butterflies run in registers and
// only the exchanges between two stages go through LDS (one write and one
// read per element and exchange, where an in-place transform of data in LDS
// has one write and one read per stage besides those that bring the data
// in and out).  The caller supplies the first stage's inputs and takes the last
// stage's outputs, each in the order that its own memory accesses want.
#pragma once

#include <type_traits>

#include "common.h"

namespace stau {

// 12 = 3 x 4: four length-3 DFTs over stride 4, twiddles e^{DIR 2 pi i n k / 12},
// three length-4 DFTs
template <int DIR, typename T>
__device__ __forceinline__ void dft12(cpx<T>* v) {
  const T h = T(0.5), s = T(0.86602540378443864676372317075294);
  cpx<T> a[4][3];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
#pragma unroll
    for (int q = 0; q < 3; ++q) a[n][q] = v[n + 4 * q];
    dft3<DIR>(a[n]);
  }
  const T d = T(DIR);
  // w^{n k}: n = 1: w, w^2; n = 2: w^2, w^4; n = 3: w^3, w^6
  a[1][1] = cmul(a[1][1], mk(s, d * h));
  a[1][2] = cmul(a[1][2], mk(h, d * s));
  a[2][1] = cmul(a[2][1], mk(h, d * s));
  a[2][2] = cmul(a[2][2], mk(-h, d * s));
  a[3][1] = mul_pi<DIR>(a[3][1]);
  a[3][2] = mk(-a[3][2].x, -a[3][2].y);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cpx<T> t[4] = {a[0][k], a[1][k], a[2][k], a[3][k]};
    dft4<DIR>(t);
#pragma unroll
    for (int m = 0; m < 4; ++m) v[k + 3 * m] = t[m];
  }
}

// 16 = 4 x 4
template <int DIR, typename T>
__device__ __forceinline__ void dft16(cpx<T>* v) {
  const T c = T(0.92387953251128675612818318939679), s = T(0.38268343236508977172845998403040);
  const T h = T(0.70710678118654752440084436210485);
  const T d = T(DIR);
  cpx<T> a[4][4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[n][q] = v[n + 4 * q];
    dft4<DIR>(a[n]);
  }
  a[1][1] = cmul(a[1][1], mk(c, d * s));
  a[1][2] = cmul(a[1][2], mk(h, d * h));
  a[1][3] = cmul(a[1][3], mk(s, d * c));
  a[2][1] = cmul(a[2][1], mk(h, d * h));
  a[2][2] = mul_pi<DIR>(a[2][2]);
  a[2][3] = cmul(a[2][3], mk(-h, d * h));
  a[3][1] = cmul(a[3][1], mk(s, d * c));
  a[3][2] = cmul(a[3][2], mk(-h, d * h));
  a[3][3] = cmul(a[3][3], mk(-c, -d * s));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    cpx<T> t[4] = {a[0][k], a[1][k], a[2][k], a[3][k]};
    dft4<DIR>(t);
#pragma unroll
    for (int m = 0; m < 4; ++m) v[k + 4 * m] = t[m];
  }
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_any(cpx<T>* v) {
  if constexpr (R == 12) dft12<DIR>(v);
  else if constexpr (R == 16) dft16<DIR>(v);
  else if constexpr (R > 1) dftR<R, DIR>(v);
}

template <int... R>
struct FftPlan;
template <>
struct FftPlan<> {};
template <typename P, int... R>
struct FftReverse {
  using type = P;
};

// The radices of a transform's stages, in order.
template <int... R>
struct FftPlan {
  static constexpr int n = sizeof...(R), r[n] = {R...}, L = (R * ...), PT = r[n - 1];
  static constexpr int ns(int s) { return s == 0 ? 1 : ns(s - 1) * r[s - 1]; }
  using reverse = typename FftReverse<FftPlan<>, R...>::type;
  // most butterflies of a stage
  static constexpr int width() {
    int w = 0;
    for (int s = 0; s < n; ++s) w = L / r[s] > w ? L / r[s] : w;
    return w;
  }
};

template <int... D, int R0, int... R>
struct FftReverse<FftPlan<D...>, R0, R...> : FftReverse<FftPlan<R0, D...>, R...> {};

template <int I, int N, typename F>
__device__ __forceinline__ void static_for_stage(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for_stage<I + 1, N>(f);
  }
}

// Butterfly index bf -> (sequence, j): sequences fastest, or j fastest
template <int B, int W, bool SF>
__device__ __forceinline__ void fft_map(int bf, int& s, int& j) {
  if constexpr (SF) {
    j = bf / B;
    s = bf - j * B;
  } else {
    s = bf / W;
    j = bf - s * W;
  }
}

// One stage: inputs of butterfly (s, j) are the elements j + r M / R, r < R; its
// outputs the elements (j / NS) NS R + j mod NS + r NS.  tw[t] = e^{-2 pi i t / M}.
template <int M, int R, int NS, int DIR, typename T>
__device__ __forceinline__ void fft_butterfly(cpx<T>* v, int j, const cpx<T>* __restrict__ tw) {
  if constexpr (NS > 1) {
    // powers from the table's entries 1 and 8 (at most three products deep)
    cpx<T> w[R > 8 ? 9 : R];
    const int t = (j % NS) * (M / (NS * R));
    w[1] = tw[t];
    if constexpr (R > 2) w[2] = cmul(w[1], w[1]);
    if constexpr (R > 3) w[3] = cmul(w[1], w[2]);
    if constexpr (R > 4) w[4] = cmul(w[2], w[2]);
#pragma unroll
    for (int r = 5; r < R && r < 8; ++r) w[r] = cmul(w[r - 4], w[4]);
    if constexpr (R > 8) w[8] = tw[8 * t];
#pragma unroll
    for (int r = 1; r < R; ++r) {
      if (r >= 8) v[r] = DIR < 0 ? cmul(v[r], w[8]) : cmulc(v[r], w[8]);
      if (r != 8) v[r] = DIR < 0 ? cmul(v[r], w[r & 7]) : cmulc(v[r], w[r & 7]);
    }
  }
  dft_any<R, DIR>(v);
}

// B transforms of the plan PL by NT threads.  load(b, s, j, v) fills the first
// stage's inputs (b counts the thread's butterflies), store(s, j, v) takes the
// last stage's outputs (elements j + r M / R of sequence s); without LAST the
// last stage is left to the caller, its inputs in LDS.  at(s, i): LDS place of
// element i.  SF0, SFL: sequences fastest over the threads in the first and last
// stage (the stages between follow the last).
template <typename PL, int DIR, int B, int NT, bool SF0, bool SFL, bool LAST, typename T, typename LD, typename ST,
          typename AT>
__device__ __forceinline__ void fft_block(cpx<T>* buf, const cpx<T>* __restrict__ tw, int tid, LD&& load, ST&& store,
                                          AT&& at) {
  constexpr int M = PL::L, NST = PL::n;
  static_for_stage<0, LAST ? NST : NST - 1>([&](auto sc) {
    constexpr int S = decltype(sc)::value;
    constexpr int R = PL::r[S], NS = PL::ns(S), W = M / R, NB = (B * W + NT - 1) / NT;
    constexpr bool SF = S == 0 ? SF0 : SFL, whole = NB * NT == B * W;
    cpx<T> v[NB][R];
    if (S > 0) __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int bf = tid + b * NT;
      if (whole || bf < B * W) {
        int s, j;
        fft_map<B, W, SF>(bf, s, j);
        if constexpr (S == 0) {
          load(b, s, j, v[b]);
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) v[b][r] = buf[at(s, j + r * W)];
        }
      }
    }
    if (S > 0 && S + 1 < NST) __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int bf = tid + b * NT;
      if (whole || bf < B * W) {
        int s, j;
        fft_map<B, W, SF>(bf, s, j);
        fft_butterfly<M, R, NS, DIR, T>(v[b], j, tw);
        if constexpr (S + 1 == NST) {
          store(s, j, v[b]);
        } else {
          const int o = (j / NS) * NS * R + j % NS;
#pragma unroll
          for (int r = 0; r < R; ++r) buf[at(s, o + r * NS)] = v[b][r];
        }
      }
    }
  });
  if constexpr (!LAST) __syncthreads();
}

}  // namespace stau
