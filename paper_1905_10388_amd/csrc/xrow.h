// Real-row transforms of the FP64 x passes at compile-time row lengths L = 3 Nx / 2,
// from registers to registers: NR rows per block, PT = the last radix, L / PT
// threads per row, up to NB2 pairs of real fields at a time, each as one complex
// sequence.  The forward transforms run the backward stages in reverse:
//   * first backward stage, radix R0 = 3 Q: butterfly j takes the entries
//     j + r W (W = L / R0).  Those of the middle third are the padding, known to
//     be zero; those of the upper third are the conjugate-symmetric partners of
//     the lower third's entries of butterfly W - j, so a thread that does both
//     butterflies reads every entry of the half spectra once;
//   * last backward stage: a thread owns the grid points j + r L / PT, r < PT, of its
//     row for every pair, forms the products there and starts the forward
//     transforms, whose first radix is PT too, from them;
//   * last forward stage: butterflies j and W - j again hold each entry and its
//     partner, so the two real fields of a sequence separate in registers; the
//     dropped third is never formed.
// Between two stages a sequence goes through LDS once.  The stages between the
// ends are spread over the block by (row, pair, butterfly).
#pragma once

#include "fft.h"
#include "xform.h"

namespace stau {

// The two half spectra of a pair (B null: one), i kx times where da, db; w0: weight
// of the entry k = 0
struct XSrc {
  const double2 *A, *B;
  bool da, db;
  double w0;
};
// Where a sequence's two spectra go (B null: one), times s0 (k = 0) or s1
struct XDst {
  double2 *A, *B;
  double s0, s1;
};

template <typename PL, int NR_, int NB2_>
struct XRow {
  using T = double;
  using cT = cpx<T>;
  static constexpr int NR = NR_, NB2 = NB2_, L = PL::L, PT = PL::PT, TR = L / PT, R0 = PL::r[0], Q = R0 / 3,
                       W = L / R0, U = W / 2, Pa = L / 3, NST = PL::n, NT = (NR * TR + 63) / 64 * 64;
  // sequence length in LDS: at radix 12 one entry of padding per 12 (the first
  // stage's writes are R0 entries apart)
  static constexpr int LS = R0 == 12 ? L / 12 * 13 : L;
  static constexpr size_t lds = (size_t)NR * NB2 * LS * sizeof(double2);
  cT* buf;  // [row][sequence][LS]
  const cT* tw;
  double kx1;  // 2 pi / Lx
  int tid, nrow, row, tj;
  bool on;

  __device__ __forceinline__ XRow(void* smem, const XformArgs& a, int nrow_)
      : buf((cT*)smem), tw((const cT*)a.twx), kx1(a.two_pi_over_Lx), tid(threadIdx.x), nrow(nrow_),
        row((int)threadIdx.x / TR), tj((int)threadIdx.x - (int)threadIdx.x / TR * TR) {
    on = row < nrow;
  }
  // LDS places: backward padded by R0 = 12; forward the low three bits of the
  // index exchanged with the next three (the first stage writes PT apart)
  static __device__ __forceinline__ int atb(int i) { return R0 == 12 ? i + i / 12 : i; }
  static __device__ __forceinline__ int atf(int i) { return i ^ ((i >> 3) & 7); }
  // (by value: a choice between two elements of register arrays by reference
  // would put both arrays into scratch memory)
  static __device__ __forceinline__ cT sel(bool c, cT x, cT y) { return mk<T>(c ? x.x : y.x, c ? x.y : y.y); }
  __device__ __forceinline__ cT ik(int k, cT c) const {
    const T kx = kx1 * (double)k;
    return mk<T>(-kx * c.y, kx * c.x);
  }

  // stages 1 .. NST - 2 of the backward (DIR +1) or forward transform of NC sequences per row
  template <int DIR, int NC>
  __device__ __forceinline__ void middle() {
    static_for_stage<1, NST - 1>([&](auto sc) __attribute__((always_inline)) {
      constexpr int S = decltype(sc)::value;
      constexpr int RS = DIR > 0 ? PL::r[S] : PL::r[NST - 1 - S], WS = L / RS;
      constexpr int NS = [] {
        int p = 1;
        for (int q = 0; q < S; ++q) p *= DIR > 0 ? PL::r[q] : PL::r[NST - 1 - q];
        return p;
      }();
      constexpr int IT = NR * NC * WS, NB = (IT + NT - 1) / NT;
      cT v[NB][RS];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int it = tid + b * NT, sq = it / WS, j = it - sq * WS;
        const cT* B = buf + ((sq / NC) * NB2 + sq % NC) * LS;
        if (IT % NT == 0 || it < IT) {
#pragma unroll
          for (int q = 0; q < RS; ++q) v[b][q] = B[DIR > 0 ? atb(j + q * WS) : atf(j + q * WS)];
        }
      }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int it = tid + b * NT, sq = it / WS, j = it - sq * WS;
        cT* B = buf + ((sq / NC) * NB2 + sq % NC) * LS;
        if (IT % NT == 0 || it < IT) {
          fft_butterfly<L, RS, NS, DIR, T>(v[b], j, tw);
          const int o = (j / NS) * NS * RS + j % NS;
#pragma unroll
          for (int q = 0; q < RS; ++q) B[DIR > 0 ? atb(o + q * NS) : atf(o + q * NS)] = v[b][q];
        }
      }
      __syncthreads();
    });
  }

  // backward transforms of NC pairs per row, src(row, i): pair i; take(i, v): the
  // PT grid points of pair i (a constant), real and imaginary parts its two fields
  template <int NC, typename SRC, typename TAKE>
  __device__ __forceinline__ void backward(SRC&& src, TAKE&& take) {
    constexpr int IT = NR * NC * U, NB = (IT + NT - 1) / NT;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int it = tid + b * NT, sq = it / U, t = it - sq * U, rw = sq / NC, p = sq % NC;
      if (rw >= nrow) continue;
      const int j1 = t, j2 = t ? W - t : U;
      cT* B = buf + (rw * NB2 + p) * LS;
      const XSrc g = src(rw, p);
      cT a1[Q], a2[Q], b1[Q], b2[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        a1[q] = ldv<T>(g.A + j1 + q * W);
        a2[q] = ldv<T>(g.A + j2 + q * W);
        b1[q] = b2[q] = mk<T>(0, 0);
        if (g.B) {
          b1[q] = ldv<T>(g.B + j1 + q * W);
          b2[q] = ldv<T>(g.B + j2 + q * W);
        }
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (g.da) {
          a1[q] = ik(j1 + q * W, a1[q]);
          a2[q] = ik(j2 + q * W, a2[q]);
        }
        if (g.db) {
          b1[q] = ik(j1 + q * W, b1[q]);
          b2[q] = ik(j2 + q * W, b2[q]);
        }
      }
      if (t == 0) {  // k = 0: real
        a1[0] = mk<T>(g.w0 * a1[0].x, 0);
        b1[0] = mk<T>(g.w0 * b1[0].x, 0);
      }
      cT v[R0];
      // entries of butterfly j1: the lower third from (a1, b1), the upper third
      // the partners of the lower one's entries of j2 (j1 = 0: its own)
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        v[q] = mk<T>(a1[q].x - b1[q].y, a1[q].y + b1[q].x);
        v[Q + q] = mk<T>(0, 0);
        const cT c2 = mk<T>(a2[q].x + b2[q].y, -a2[q].y + b2[q].x);
        cT n1 = mk<T>(0, 0);  // (j1 = 0: k = (q + 1) W, padding for q = Q - 1)
        if constexpr (Q > 1) {
          if (q + 1 < Q) n1 = mk<T>(a1[(q + 1) % Q].x + b1[(q + 1) % Q].y, -a1[(q + 1) % Q].y + b1[(q + 1) % Q].x);
        }
        v[R0 - 1 - q] = sel(t, c2, n1);
      }
      dft_any<R0, +1>(v);
#pragma unroll
      for (int q = 0; q < R0; ++q) B[atb(j1 * R0 + q)] = v[q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        v[q] = mk<T>(a2[q].x - b2[q].y, a2[q].y + b2[q].x);
        v[Q + q] = mk<T>(0, 0);
        const cT c1 = mk<T>(a1[q].x + b1[q].y, -a1[q].y + b1[q].x), c2 = mk<T>(a2[q].x + b2[q].y, -a2[q].y + b2[q].x);
        v[R0 - 1 - q] = sel(t, c1, c2);
      }
      dft_any<R0, +1>(v);
#pragma unroll
      for (int q = 0; q < R0; ++q) B[atb(j2 * R0 + q)] = v[q];
    }
    __syncthreads();
    middle<+1, NC>();
    if (on) {
      static_for_stage<0, NC>([&](auto pc) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
        const cT* B = buf + (row * NB2 + p) * LS;
        cT v[PT];
#pragma unroll
        for (int q = 0; q < PT; ++q) v[q] = B[atb(tj + q * TR)];
        fft_butterfly<L, PT, L / PT, +1, T>(v, tj, tw);
        take(pc, v);
      });
    }
    __syncthreads();
  }

  // forward transforms of NC sequences per row: give(i, v) supplies the PT grid
  // points of sequence i (a constant), dst(row, i) its two spectra's places
  template <int NC, typename GIVE, typename DST>
  __device__ __forceinline__ void forward(GIVE&& give, DST&& dst) {
    if (on) {
      static_for_stage<0, NC>([&](auto pc) __attribute__((always_inline)) {
        constexpr int p = decltype(pc)::value;
        cT* B = buf + (row * NB2 + p) * LS;
        cT v[PT];
        give(pc, v);
        dft_any<PT, -1>(v);
#pragma unroll
        for (int q = 0; q < PT; ++q) B[atf(tj * PT + q)] = v[q];
      });
    }
    __syncthreads();
    middle<-1, NC>();
    constexpr int IT = NR * NC * U, NB = (IT + NT - 1) / NT;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int it = tid + b * NT, sq = it / U, t = it - sq * U, rw = sq / NC, p = sq % NC;
      if (rw >= nrow) continue;
      const int j1 = t, j2 = t ? W - t : U;
      const cT* B = buf + (rw * NB2 + p) * LS;
      cT v1[R0], v2[R0];
#pragma unroll
      for (int q = 0; q < R0; ++q) {
        v1[q] = B[atf(j1 + q * W)];
        v2[q] = B[atf(j2 + q * W)];
      }
      fft_butterfly<L, R0, W, -1, T>(v1, j1, tw);
      fft_butterfly<L, R0, W, -1, T>(v2, j2, tw);
      const XDst h = dst(rw, p);
      auto put = [&](int k, T sc, cT z, cT m) __attribute__((always_inline)) {
        stv<T>(h.A + k, mk<T>(sc * (z.x + m.x), sc * (z.y - m.y)));
        if (h.B) stv<T>(h.B + k, mk<T>(sc * (z.y + m.y), -sc * (z.x - m.x)));
      };
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        // partner L - k of k = j + q W
        put(j1 + q * W, q == 0 && t == 0 ? h.s0 : h.s1, v1[q], sel(t, v2[R0 - 1 - q], v1[q ? R0 - q : 0]));
        put(j2 + q * W, h.s1, v2[q], sel(t, v1[R0 - 1 - q], v2[R0 - 1 - q]));
      }
      if (t == 0) {  // Nyquist slot
        stv<T>(h.A + Pa, mk<T>(0, 0));
        if (h.B) stv<T>(h.B + Pa, mk<T>(0, 0));
      }
    }
    __syncthreads();
  }
};

}  // namespace stau
