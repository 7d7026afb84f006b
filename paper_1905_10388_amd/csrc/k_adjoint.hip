// Adjoint transform kernels of the discrete adjoint step: the transposes of
// the z transforms, of the fused x pass and of the kinetic-energy and
// initial-state maps.
#include "xrow.h"

namespace stau {

// ===========================================================================
// Adjoint kernels.  Complex coefficients are pairs of independent reals; the
// adjoint of z is dJ/dRe z + i dJ/dIm z.  Real-grid adjoints are real.
// ===========================================================================

// Adjoint of the backward z transform (c -> g_j = sum_n c_n T_n(z_j), with
// c optionally multiplied by i k): c_bar_n += conj(i k) sum_j T_n(z_j) g_bar_j,
// i.e. an unweighted DCT-II per source field, summed per target variable and
// accumulated into Xbar[p][var][n].
template <int MAXBF, int MAXIT, typename T, int EPT = kZEpt>
__global__ void __launch_bounds__(kZThreads) zadj_kernel(XformArgs a, AccList al,
                                                         const typename V2<T>::type* __restrict__ Gb,
                                                         double2* __restrict__ Xb, int TP) {
  extern __shared__ double2 smem[];
  using cT = cpx<T>;
  const int M = a.M, N = a.N, S = a.S;
  cT* buf = (cT*)smem;
  cT* twl = buf + EPT * kZThreads;  // FFT twiddles after the EPT * kZThreads tile points
  cT* dcl = twl + M;
  const int ti = blockIdx.y;
  const int p0 = blockIdx.x * TP;
  const int tid = threadIdx.x, nt = kZThreads;
  stage_z_tables<T>(a, twl, dcl, M, tid);
  cd acc[MAXIT];
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) acc[it] = mk(0.0, 0.0);
  for (int q = 0; q < al.nsrc[ti]; ++q) {
    const int f = al.src[ti][q], der = al.deriv[ti][q];
    {
      cT hv[EPT];
#pragma unroll
      for (int it = 0; it < EPT; ++it) {
        const int idx = tid + it * nt;
        const int jz = idx / TP, s = idx - jz * TP;
        const int p = p0 + s;
        hv[it] = mk<T>(0, 0);
        if (p < a.P) hv[it] = ldv<T>(Gb + ((size_t)f * M + jz) * a.P + p);
      }
#pragma unroll
      for (int it = 0; it < EPT; ++it) {
        const int idx = tid + it * nt;
        const int jz = idx / TP, s = idx - jz * TP;
        const int dst = (jz & 1) ? (M - 1 - (jz >> 1)) : (jz >> 1);
        buf[s * M + dst] = hv[it];
      }
    }
    __syncthreads();
    fft_lds<-1, MAXBF>(buf, M, TP, (const cT*)twl, tid, nt);
#pragma unroll
    for (int it = 0; it < MAXIT; ++it) {
      const int idx = tid + it * nt;
      if (idx < TP * N) {
        const int s = idx / N, nn = idx - s * N;
        const int p = p0 + s;
        const cT V = buf[s * M + nn];
        const cT Vm = buf[s * M + (nn == 0 ? 0 : M - nn)];
        const cT w = conj(dcl[nn]);
        const cT P = cmul(w, V), Q = cmul(w, conj(Vm));
        cd Y = mk((double)((T)0.5 * (P.x + Q.x)), (double)((T)0.5 * (P.y - Q.y)));
        if (nn & 1) Y = mk(-Y.x, -Y.y);
        if (der && p < a.P) {
          const double kk = der == 1 ? kx_of(a, p) : ky_of(a, p);
          Y = mk(kk * Y.y, -kk * Y.x);  // conj(i k) Y = -i k Y
        }
        acc[it] = acc[it] + Y;
      }
    }
    __syncthreads();
  }
  const int var = al.target[ti];
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int idx = tid + it * nt;
    if (idx < TP * N) {
      const int s = idx / N, nn = idx - s * N;
      const int p = p0 + s;
      if (active(a, p)) {
        double2* o = Xb + ((size_t)p * S + var) * N + nn;
        const double2 old = *o;
        *o = make_double2(old.x + acc[it].x, old.y + acc[it].y);
      }
    }
  }
}

// Adjoint of the fused x pass for one dealiased z row.  Recomputes the eight
// forward grid fields from G, maps the explicit-term adjoints H_bar to the
// grid (adjoint of the truncated real-to-complex transform:
// g_bar_i = (1/L) [Re c_0 + Re sum_{k>=1} c_k e^{2 pi i k i / L}]), applies the
// product rule, and maps the eight grid adjoints back to spectra (adjoint of
// the complex-to-real synthesis: c_bar_k = w_k sum_i g_bar_i e^{-2 pi i k i/L},
// w_0 = 1, w_k = 2).  SPLIT: two blocks per row (blockIdx.y 0: the (u, w)
// outputs, 1: the derivative outputs), for launches with fewer rows than
// compute units; each block synthesises the fields its outputs need.
template <int MAXBF, int PTS, int NT, bool TWL, typename T, bool SPLIT>
__global__ void __launch_bounds__(NT) xpass_adj_kernel(XformArgs a,
                                                       const typename V2<T>::type* __restrict__ G,
                                                       const typename V2<T>::type* __restrict__ Hb,
                                                       typename V2<T>::type* __restrict__ Gb) {
  extern __shared__ double2 smem[];
  using cT = cpx<T>;
  using S2 = typename V2<T>::type;
  constexpr int KPT = (PTS + 2) / 3;  // half-spectrum entries per thread (Pa = L / 3)
  cT* buf = (cT*)smem;
  const int jz = blockIdx.x;
  const int M = a.M, L = a.L, Pa = a.Pa, P = a.P;
  const int tid = threadIdx.x;
  const cT* twg = (const cT*)(sizeof(T) == 8 ? (const void*)a.twx : (const void*)a.twx32);
  cT* twl = buf + L;
  if constexpr (TWL) {
    for (int i = tid; i < L; i += NT) twl[i] = twg[i];
  }
  const cT* tw = TWL ? (const cT*)twl : twg;
  auto row = [&](const S2* base, int f) { return base + ((size_t)f * M + jz) * P; };
  // complex-to-real pairs: 0..3 the forward fields (G 0..7), 4 (Hb 0, Hb 1)
  // and 5 (Hb 2, -); hs scales k >= 1 (1 for synthesis, 0.5 for the adjoint
  // of the truncated forward transform)
  cT sa[KPT], sb[KPT];
  auto fetch = [&](int k) {
    const S2* A = k < 4 ? row(G, 2 * k) : row(Hb, 2 * (k - 4));
    const S2* B = k < 4 ? row(G, 2 * k + 1) : (k == 4 ? row(Hb, 1) : nullptr);
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      const int kk = tid + q * NT;
      sa[q] = mk<T>(0, 0);
      sb[q] = mk<T>(0, 0);
      if (kk < Pa) {
        sa[q] = ldv<T>(A + kk);
        if (B) sb[q] = ldv<T>(B + kk);
      }
    }
  };
  auto scatter = [&](T hs) {
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      const int kk = tid + q * NT;
      if (kk < Pa) {
        cT Ak = sa[q], Bk = sb[q];
        if (kk == 0) {
          Ak.y = 0;
          Bk.y = 0;
        } else {
          Ak = scale(Ak, hs);
          Bk = scale(Bk, hs);
        }
        buf[kk] = mk<T>(Ak.x - Bk.y, Ak.y + Bk.x);
        if (kk > 0) buf[L - kk] = mk<T>(Ak.x + Bk.y, -Ak.y + Bk.x);
      }
    }
    for (int k = Pa + tid; k <= L - Pa; k += NT) buf[k] = mk<T>(0, 0);
  };
  // adjoint of a synthesis pair: spectra of two real grid rows, weights w_k
  auto r2c_adj_pair = [&](const T* ga, const T* gb, int fa, int fb) {
#pragma unroll
    for (int q = 0; q < PTS; ++q) {
      const int i = tid + q * NT;
      if (i < L) buf[i] = mk<T>(ga[q], gb[q]);
    }
    __syncthreads();
    fft_lds<-1, MAXBF, T, true>(buf, L, 1, tw, tid, NT);
    S2* Oa = Gb + ((size_t)fa * M + jz) * P;
    S2* Ob = Gb + ((size_t)fb * M + jz) * P;
    for (int k = tid; k < P; k += NT) {
      cT A = mk<T>(0, 0), Bv = mk<T>(0, 0);
      if (k < Pa) {
        const cT Zk = buf[k], Zm = buf[k == 0 ? 0 : L - k];
        const T wk = k == 0 ? (T)1 : (T)2;
        A = mk<T>((T)0.5 * (Zk.x + Zm.x) * wk, (T)0.5 * (Zk.y - Zm.y) * wk);
        Bv = mk<T>((T)0.5 * (Zk.y + Zm.y) * wk, (T)-0.5 * (Zk.x - Zm.x) * wk);
      }
      stv<T>(Oa + k, A);
      stv<T>(Ob + k, Bv);
    }
    __syncthreads();
  };

  // The grid fields are consumed as they are synthesised: the explicit-term
  // adjoints first (n_b, n_u, n_w), then the derivative pairs accumulate the
  // (u, w) adjoints t1 = -(n . grad_x), t2 = -(n . grad_z), and (u, w) feeds
  // the derivative adjoints -n_q (u, w).  Part 1 computes the (u, w) outputs,
  // part 2 the six derivative outputs (blocks of a split launch), part 0 both.
  auto body = [&](auto part_c) {
    constexpr int PART = decltype(part_c)::value;
    constexpr int NS = PART == 1 ? 5 : PART == 2 ? 3 : 6;
    // synthesis order: 4, 5 (H_bar), then part 1: 1, 2, 3; part 2: 0; part 0: 1, 2, 3, 0
    auto seq = [](int i) { return i == 0 ? 4 : i == 1 ? 5 : PART == 2 ? 0 : i < 5 ? i - 1 : 0; };
    T u[PTS], w[PTS], nb[PTS], nu[PTS], nw[PTS], t1[PTS], t2[PTS];
    const T invL = (T)1 / (T)L;
    fetch(seq(0));
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int k = seq(i);
      scatter(k < 4 ? (T)1 : (T)0.5);
      if (i + 1 < NS) fetch(seq(i + 1));
      __syncthreads();
      fft_lds<+1, MAXBF, T, true>(buf, L, 1, tw, tid, NT);
#pragma unroll
      for (int q = 0; q < PTS; ++q) {
        const int ii = tid + q * NT;
        if (ii < L) {
          const T x = buf[ii].x, y = buf[ii].y;
          if (k == 4) {
            nb[q] = x * invL;
            nu[q] = y * invL;
          } else if (k == 5) {
            nw[q] = x * invL;
          } else if (k == 0) {
            u[q] = x;
            w[q] = y;
          } else if (k == 1) {
            t1[q] = -(nb[q] * x);
            t2[q] = -(nb[q] * y);
          } else {
            const T n = k == 2 ? nu[q] : nw[q];
            t1[q] -= n * x;
            t2[q] -= n * y;
          }
        }
      }
      __syncthreads();
    }
    if constexpr (PART != 2) r2c_adj_pair(t1, t2, 0, 1);
    if constexpr (PART != 1) {
#pragma unroll
      for (int q = 0; q < PTS; ++q) {
        t1[q] = -nb[q] * u[q];
        t2[q] = -nb[q] * w[q];
      }
      r2c_adj_pair(t1, t2, 2, 3);
#pragma unroll
      for (int q = 0; q < PTS; ++q) {
        t1[q] = -nu[q] * u[q];
        t2[q] = -nu[q] * w[q];
      }
      r2c_adj_pair(t1, t2, 4, 5);
#pragma unroll
      for (int q = 0; q < PTS; ++q) {
        t1[q] = -nw[q] * u[q];
        t2[q] = -nw[q] * w[q];
      }
      r2c_adj_pair(t1, t2, 6, 7);
    }
  };
  if constexpr (SPLIT) {
    if (blockIdx.y == 0)
      body(std::integral_constant<int, 1>{});
    else
      body(std::integral_constant<int, 2>{});
  } else {
    body(std::integral_constant<int, 0>{});
  }
}

// The same in FP64 at the compile-time row lengths (XRow), always two blocks per
// row: blockIdx.y 0 synthesises H_bar and the derivative pairs for the (u, w)
// outputs, 1 synthesises H_bar and (u, w) for the derivative outputs.  Bound by
// its chain of transforms (adjoint step with this and zadj_fft_kernel against
// the in-place kernels: 512x128 120 -> 97 us, 4096x32 192 -> 144, 256x64 90 -> 65;
// the transposed solve has 56 of the 97).
template <typename PL, int NB2, int WPE>
__global__ void __launch_bounds__((XRow<PL, 1, NB2>::NT)) __attribute__((amdgpu_waves_per_eu(WPE)))
    xadj_fft_kernel(XformArgs a, const double2* __restrict__ G, const double2* __restrict__ Hb,
                    double2* __restrict__ Gb) {
  extern __shared__ double2 smem[];
  using X = XRow<PL, 1, NB2>;
  using T = double;
  using cT = cpx<T>;
  constexpr int PT = X::PT, P = X::Pa + 1;
  X x(smem, a, 1);
  const size_t row = (size_t)blockIdx.x * P, R = (size_t)a.M * P;
  // pairs 0..3 the forward fields (G 0..7), 4 (Hb 0, Hb 1) and 5 (Hb 2, -): these
  // with weight 1/2 for k >= 1, here 2 for k = 0 and 1/2 in hf
  auto pair = [&](int k) {
    if (k < 4) return XSrc{G + row + 2 * k * R, G + row + (2 * k + 1) * R, false, false, 1.0};
    return XSrc{Hb + row + 2 * (k - 4) * R, k == 4 ? Hb + row + R : nullptr, false, false, 2.0};
  };
  const T hf = (T)0.5 / (T)X::L;
  T nb[PT], nu[PT], nw[PT], s[PT], t[PT];  // s, t: the (u, w) adjoints, or u and w
  // pair K of one or two transformed together
  auto take = [&](auto kc, const cT* v) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value;
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const T f = v[q].x, g = v[q].y;
      if (K == 0) { s[q] = f; t[q] = g; }
      if (K == 1) { s[q] = -(nb[q] * f); t[q] = -(nb[q] * g); }
      if (K == 2) { s[q] -= nu[q] * f; t[q] -= nu[q] * g; }
      if (K == 3) { s[q] -= nw[q] * f; t[q] -= nw[q] * g; }
      if (K == 4) { nb[q] = hf * f; nu[q] = hf * g; }
      if (K == 5) nw[q] = hf * f;
    }
  };
  auto run1 = [&](auto kc) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value;
    x.template backward<1>([&](int, int) { return pair(K); },
                           [&](auto, const cT* v) __attribute__((always_inline)) { take(kc, v); });
  };
  auto run2 = [&](auto k0, auto k1) __attribute__((always_inline)) {
    constexpr int K0 = decltype(k0)::value, K1 = decltype(k1)::value;
    if constexpr (NB2 >= 2) {
      x.template backward<2>([&](int, int p) { return pair(p ? K1 : K0); },
                             [&](auto pc, const cT* v) __attribute__((always_inline)) {
                               take(std::integral_constant<int, decltype(pc)::value ? K1 : K0>{}, v);
                             });
    } else {
      run1(k0);
      run1(k1);
    }
  };
  // adjoint of a synthesis: weights 1 (k = 0) and 2
  auto out = [&](int f) { return XDst{Gb + row + f * R, Gb + row + (f + 1) * R, 0.5, 1.0}; };
  auto deriv = [&](auto fc, cT* v) __attribute__((always_inline)) {  // outputs -n_f (u, w)
    constexpr int F = decltype(fc)::value;
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const T n = F == 0 ? nb[q] : F == 1 ? nu[q] : nw[q];
      v[q] = mk<T>(-n * s[q], -n * t[q]);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;
  using I5 = std::integral_constant<int, 5>;
  run2(I4{}, I5{});
  if (blockIdx.y == 0) {
    run2(I1{}, I2{});
    run1(I3{});
    x.template forward<1>(
        [&](auto, cT* v) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < PT; ++q) v[q] = mk<T>(s[q], t[q]);
        },
        [&](int, int) { return out(0); });
  } else {
    run1(I0{});
    if constexpr (NB2 >= 2) {
      x.template forward<2>([&](auto pc, cT* v) __attribute__((always_inline)) { deriv(pc, v); },
                            [&](int, int p) { return out(2 + 2 * p); });
    } else {
      x.template forward<1>([&](auto, cT* v) __attribute__((always_inline)) { deriv(I0{}, v); },
                            [&](int, int) { return out(2); });
      x.template forward<1>([&](auto, cT* v) __attribute__((always_inline)) { deriv(I1{}, v); },
                            [&](int, int) { return out(4); });
    }
    x.template forward<1>([&](auto, cT* v) __attribute__((always_inline)) { deriv(I2{}, v); },
                          [&](int, int) { return out(6); });
  }
}

// The z adjoint in FP64 at the dealiased lengths (as zf_fft_kernel): a thread's two
// last-stage butterflies hold V_n and V_{M-n}, their sum over the sources stays in
// registers.
template <typename PL, int TP, int NT>
__global__ void __launch_bounds__(NT) zadj_fft_kernel(XformArgs a, AccList al, const double2* __restrict__ Gb,
                                                      double2* __restrict__ Xb) {
  extern __shared__ double2 smem[];
  constexpr int M = PL::L, N = M / 3 * 2, R0 = PL::r[0], W0 = M / R0, RL = PL::PT, W = M / RL, U = W / 2,
                QN = RL / 3 * 2;
  static_assert(RL % 3 == 0 && TP * U <= NT, "thirds of the last stage, one pair of butterflies per thread");
  cd* buf = (cd*)smem;
  const int ti = blockIdx.y, p0 = blockIdx.x * TP, tid = threadIdx.x;
  const PencilBase pb = pencil_base(a, p0);
  auto at = [](int s, int i) { return s * (M + 1) + i; };
  auto sel = [](bool c, cd x, cd y) { return mk(c ? x.x : y.x, c ? x.y : y.y); };
  const int s0 = tid % TP, t = tid / TP;
  const bool own = t < U;
  const int j1 = t, j2 = t ? W - t : U;
  cd acc1[QN], acc2[QN];
#pragma unroll
  for (int q = 0; q < QN; ++q) acc1[q] = acc2[q] = mk(0.0, 0.0);
  for (int src = 0; src < al.nsrc[ti]; ++src) {
    const int f = al.src[ti][src], der = al.deriv[ti][src];
    auto load = [&](int, int s, int j, cd* v) {
      const double2* h = Gb + (size_t)f * M * a.P + p0 + s;
      const bool in = p0 + s < a.P;
#pragma unroll
      for (int q = 0; q < R0; ++q) {
        const int i = j + q * W0, jz = 2 * i < M ? 2 * i : 2 * (M - 1 - i) + 1;
        v[q] = in ? ld2(h + (size_t)jz * a.P) : mk(0.0, 0.0);
      }
    };
    fft_block<PL, -1, TP, NT, true, true, false, double>(buf, (const cd*)a.twz, tid, load, [](int, int, cd*) {}, at);
    if (own) {
      cd v1[RL], v2[RL];
#pragma unroll
      for (int q = 0; q < RL; ++q) {
        v1[q] = buf[at(s0, j1 + q * W)];
        v2[q] = buf[at(s0, j2 + q * W)];
      }
      fft_butterfly<M, RL, W, -1, double>(v1, j1, (const cd*)a.twz);
      fft_butterfly<M, RL, W, -1, double>(v2, j2, (const cd*)a.twz);
      const double kk = der == 0 ? 0.0 : der == 1 ? kx_at(a, pb, s0) : ky_at(a, pb, s0);
      auto add = [&](cd& acc, int n, cd V, cd Vm) {
        const cd w = conj(ld2(a.dctz + n));
        const cd P = cmul(w, V), Q = cmul(w, conj(Vm));
        const double sc = n & 1 ? -0.5 : 0.5;
        cd Y = mk(sc * (P.x + Q.x), sc * (P.y - Q.y));
        if (der) Y = mk(kk * Y.y, -kk * Y.x);  // conj(i k) Y = -i k Y
        acc = acc + Y;
      };
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        add(acc1[q], j1 + q * W, v1[q], sel(t, v2[RL - 1 - q], v1[q ? RL - q : 0]));
        add(acc2[q], j2 + q * W, v2[q], sel(t, v1[RL - 1 - q], v2[RL - 1 - q]));
      }
    }
    __syncthreads();
  }
  if (own) {
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      buf[at(s0, j1 + q * W)] = acc1[q];
      buf[at(s0, j2 + q * W)] = acc2[q];
    }
  }
  __syncthreads();
  const int var = al.target[ti];
#pragma unroll 4
  for (int idx = tid; idx < TP * N; idx += NT) {
    const int s = idx / N, nn = idx - s * N;
    if (active_at(a, pb, s)) {
      double2* o = Xb + ((size_t)(p0 + s) * a.S + var) * N + nn;
      const cd v = buf[at(s, nn)];
      const double2 old = *o;
      *o = make_double2(old.x + v.x, old.y + v.y);
    }
  }
}

// Kinetic-energy adjoint for one row: u_bar = e_bar_j u, w_bar = e_bar_j w with
// e_bar_j = (1/L) sum_m w_m (2 - delta)/M T_m(z_j) (precomputed in ebar).
template <int MAXBF, int PTS, int NT>
__global__ void __launch_bounds__(NT) ke_row_adj_kernel(XformArgs a, const double2* __restrict__ G,
                                                        const double2* __restrict__ ebar,
                                                        double2* __restrict__ Gb) {
  extern __shared__ double2 smem[];
  cd* buf = (cd*)smem;
  const int jz = blockIdx.x;
  const int M = a.M, L = a.L, Pa = a.Pa, P = a.P;
  const int tid = threadIdx.x;
  constexpr int nt = NT;
  const cd* tw = (const cd*)a.twx;
  const double2* A = G + ((size_t)0 * M + jz) * P;
  const double2* B = G + ((size_t)1 * M + jz) * P;
  for (int k = tid; k < L; k += nt) {
    cd z = mk(0.0, 0.0);
    if (k < Pa) {
      cd Ak = ld2(A + k), Bk = ld2(B + k);
      if (k == 0) {
        Ak.y = 0.0;
        Bk.y = 0.0;
      }
      z = mk(Ak.x - Bk.y, Ak.y + Bk.x);
    } else if (k > L - Pa) {
      cd Ak = ld2(A + (L - k)), Bk = ld2(B + (L - k));
      z = mk(Ak.x + Bk.y, -Ak.y + Bk.x);
    }
    buf[k] = z;
  }
  __syncthreads();
  fft_lds<+1, MAXBF>(buf, L, 1, tw, tid, nt);
  const double e = ebar[jz].x / (double)L;
  double gu[PTS], gw[PTS];
#pragma unroll
  for (int q = 0; q < PTS; ++q) {
    const int i = tid + q * nt;
    if (i < L) {
      gu[q] = e * buf[i].x;
      gw[q] = e * buf[i].y;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PTS; ++q) {
    const int i = tid + q * nt;
    if (i < L) buf[i] = mk(gu[q], gw[q]);
  }
  __syncthreads();
  fft_lds<-1, MAXBF>(buf, L, 1, tw, tid, nt);
  double2* Oa = Gb + ((size_t)0 * M + jz) * P;
  double2* Ob = Gb + ((size_t)1 * M + jz) * P;
  for (int k = tid; k < P; k += nt) {
    cd Av = mk(0.0, 0.0), Bv = mk(0.0, 0.0);
    if (k < Pa) {
      cd Zk = buf[k], Zm = buf[k == 0 ? 0 : L - k];
      const double wk = k == 0 ? 1.0 : 2.0;
      Av = mk(0.5 * (Zk.x + Zm.x) * wk, 0.5 * (Zk.y - Zm.y) * wk);
      Bv = mk(0.5 * (Zk.y + Zm.y) * wk, -0.5 * (Zk.x - Zm.x) * wk);
    }
    st2(Oa + k, Av);
    st2(Ob + k, Bv);
  }
}

// Initial-state adjoint, step 1 (per pencil): c_bar = X_bar_b + D^T X_bar_bz
// for bz = D b, D_nm = 4 m / (1 + delta_n0) for n < m, m - n odd (d/dz on
// [0, 1] of the T-to-T derivative).
__global__ void ic_adj_coef_kernel(XformArgs a, const double2* __restrict__ Xb,
                                   double2* __restrict__ C, int vb, int vbz) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.P) return;
  const int N = a.N, S = a.S;
  const double2* xb = Xb + ((size_t)p * S + vb) * N;
  const double2* xz = Xb + ((size_t)p * S + vbz) * N;
  double2* c = C + (size_t)p * N;
  double se_r = 0.0, se_i = 0.0, so_r = 0.0, so_i = 0.0;  // running sums over even / odd n
  for (int m = 0; m < N; ++m) {
    double vr = xb[m].x, vi = xb[m].y;
    if (m & 1) {
      vr += 4.0 * m * se_r;
      vi += 4.0 * m * se_i;
    } else {
      vr += 4.0 * m * so_r;
      vi += 4.0 * m * so_i;
    }
    c[m] = make_double2(vr, vi);
    const double f = m == 0 ? 0.5 : 1.0;
    if (m & 1) {
      so_r += xz[m].x;
      so_i += xz[m].y;
    } else {
      se_r += f * xz[m].x;
      se_i += f * xz[m].y;
    }
  }
}

// Initial-state adjoint, step 3 (per z level): g_bar_i = (1/Nx) [Re H_0 +
// Re sum_{k>=1} H_k e^{2 pi i k i / Nx}] (adjoint of the truncated forward x
// transform at scale 1), written to gbar[ix][jz].
template <int MAXBF>
__global__ void __launch_bounds__(256) ic_adj_x_kernel(XformArgs a, const double2* __restrict__ H1,
                                                       double* __restrict__ gbar) {
  extern __shared__ double2 smem[];
  cd* buf = (cd*)smem;
  const int jz = blockIdx.x;
  const int Nx = a.Nx, N = a.N, Pa = a.Pa;
  const int tid = threadIdx.x, nt = blockDim.x;
  const double2* h = H1 + (size_t)jz * a.P;
  for (int k = tid; k < Nx; k += nt) {
    cd z = mk(0.0, 0.0);
    if (k == 0)
      z = mk(h[0].x, 0.0);
    else if (k < Pa)
      z = scale(ld2(h + k), 0.5);
    else if (k > Nx - Pa)
      z = scale(conj(ld2(h + (Nx - k))), 0.5);
    buf[k] = z;
  }
  __syncthreads();
  fft_lds<+1, MAXBF>(buf, Nx, 1, (const cd*)a.twx, tid, nt);
  const double inv = 1.0 / (double)Nx;
  for (int i = tid; i < Nx; i += nt) gbar[(size_t)i * N + jz] = buf[i].x * inv;
}

template <typename PL, int TP, int NT>
static hipError_t launch_zadj_fft(const XformArgs& a, const AccList& al, const void* Gbar, void* Xbar,
                                  hipStream_t st) {
  constexpr size_t lds = (size_t)TP * (PL::L + 1) * sizeof(double2);
  auto fn = zadj_fft_kernel<PL, TP, NT>;
  allow_lds((const void*)fn, lds);
  hipLaunchKernelGGL(fn, dim3((a.P + TP - 1) / TP, al.nt), dim3(NT), lds, st, a, al, (const double2*)Gbar,
                     (double2*)Xbar);
  return hipGetLastError();
}

hipError_t launch_zadj(const XformArgs& a, const AccList& al, const void* Gbar, void* Xbar,
                       hipStream_t st, bool fp32) {
  if (!fp32 && 2 * a.M == 3 * a.N) {
    const bool few = (a.P + 7) / 8 * al.nt < 2 * unit_count();  // (as in launch_zb)
    switch (a.M) {
      case 24: return launch_zadj_fft<FftPlan<4, 6>, 8, 64>(a, al, Gbar, Xbar, st);
      case 48:
        return few ? launch_zadj_fft<FftPlan<8, 6>, 4, 64>(a, al, Gbar, Xbar, st)
                   : launch_zadj_fft<FftPlan<8, 6>, 8, 64>(a, al, Gbar, Xbar, st);
      case 96:
        return few ? launch_zadj_fft<FftPlan<4, 4, 6>, 4, 64>(a, al, Gbar, Xbar, st)
                   : launch_zadj_fft<FftPlan<4, 4, 6>, 8, 128>(a, al, Gbar, Xbar, st);
      case 192:
        return few ? launch_zadj_fft<FftPlan<4, 8, 6>, 4, 128>(a, al, Gbar, Xbar, st)
                   : launch_zadj_fft<FftPlan<4, 8, 6>, 8, 128>(a, al, Gbar, Xbar, st);
      case 384:
        return few ? launch_zadj_fft<FftPlan<8, 8, 6>, 4, 256>(a, al, Gbar, Xbar, st)
                   : launch_zadj_fft<FftPlan<8, 8, 6>, 8, 256>(a, al, Gbar, Xbar, st);
      case 768: return launch_zadj_fft<FftPlan<8, 4, 4, 6>, 4, 256>(a, al, Gbar, Xbar, st);
    }
  }
  int TP = z_tile(a.M);
  if (TP * a.M != kZPts || TP * a.N > 12 * kZThreads) return hipErrorInvalidValue;
  // half-size tiles when the full-size grid has fewer blocks than compute
  // units (512x128: 102 -> 198 blocks, adjoint step 146 -> 139 us; at 4096x64,
  // 390 -> 774 blocks, half tiles measured 7 us slower)
  const int dv = z_split((a.P + TP - 1) / TP * al.nt, a.M, 1);
  TP /= dv;
  const int pts = kZPts / dv;
  dim3 grid((a.P + TP - 1) / TP, al.nt);
  auto go = [&](auto kern, auto g) {
    const size_t lds = (size_t)(pts + 2 * a.M) * sizeof(*g);
    allow_lds((const void*)kern, lds);
    hipLaunchKernelGGL(kern, grid, dim3(kZThreads), lds, st, a, al, g, (double2*)Xbar, TP);
  };
  if (fp32) {
    if (dv == 2) go(zadj_kernel<3, 12, float, kZEpt / 2>, (const float2*)Gbar);
    else go(zadj_kernel<3, 12, float>, (const float2*)Gbar);
  } else {
    if (dv == 2) go(zadj_kernel<3, 12, double, kZEpt / 2>, (const double2*)Gbar);
    else go(zadj_kernel<3, 12, double>, (const double2*)Gbar);
  }
  return hipGetLastError();
}

template <int NT, int PTS, int MAXBF, typename T>
static hipError_t launch_xpass_adj_t(const XformArgs& a, const void* G, const void* Hb, void* Gb,
                                     hipStream_t st) {
  using S2 = typename V2<T>::type;
  const bool twl = (size_t)a.L * sizeof(S2) <= 32768;
  const size_t lds = (size_t)a.L * sizeof(S2) * (twl ? 2 : 1);
  int dev = 0, cus = 0;
  const bool split = hipGetDevice(&dev) == hipSuccess &&
                     hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                     a.M < cus;
  auto go = [&](auto fn) {
    allow_lds((const void*)fn, lds);
    hipLaunchKernelGGL(fn, dim3(a.M, split ? 2 : 1), dim3(NT), lds, st, a, (const S2*)G,
                       (const S2*)Hb, (S2*)Gb);
  };
  if (twl) {
    if (split)
      go(xpass_adj_kernel<MAXBF, PTS, NT, true, T, true>);
    else
      go(xpass_adj_kernel<MAXBF, PTS, NT, true, T, false>);
  } else {
    if (split)
      go(xpass_adj_kernel<MAXBF, PTS, NT, false, T, true>);
    else
      go(xpass_adj_kernel<MAXBF, PTS, NT, false, T, false>);
  }
  return hipGetLastError();
}

template <int NB2, int WPE, int... R>
static hipError_t launch_xadj_fft(const XformArgs& a, const void* G, const void* Hb, void* Gb, hipStream_t st) {
  using X = XRow<FftPlan<R...>, 1, NB2>;
  auto fn = xadj_fft_kernel<FftPlan<R...>, NB2, WPE>;
  allow_lds((const void*)fn, X::lds);
  hipLaunchKernelGGL(fn, dim3(a.M, 2), dim3(X::NT), X::lds, st, a, (const double2*)G, (const double2*)Hb,
                     (double2*)Gb);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_xpass_adj_T(const XformArgs& a, const void* G, const void* Hb, void* Gb,
                                     hipStream_t st) {
  const int L = a.L;
  // (the radices of the x pass)
  if (sizeof(T) == 8) switch (L) {
    case 24: return launch_xadj_fft<2, 2, 6, 4>(a, G, Hb, Gb, st);
    case 48: return launch_xadj_fft<2, 2, 3, 4, 4>(a, G, Hb, Gb, st);
    case 96: return launch_xadj_fft<2, 2, 3, 8, 4>(a, G, Hb, Gb, st);
    case 192: return launch_xadj_fft<2, 2, 3, 8, 8>(a, G, Hb, Gb, st);
    case 384: return launch_xadj_fft<2, 2, 6, 8, 8>(a, G, Hb, Gb, st);
    case 768: return launch_xadj_fft<2, 2, 6, 16, 8>(a, G, Hb, Gb, st);
    case 1536: return launch_xadj_fft<2, 2, 3, 8, 8, 8>(a, G, Hb, Gb, st);
    case 3072: return launch_xadj_fft<2, 2, 6, 8, 8, 8>(a, G, Hb, Gb, st);
    case 6144: return launch_xadj_fft<1, 3, 6, 16, 8, 8>(a, G, Hb, Gb, st);
  }
  if (L <= 64) return launch_xpass_adj_t<64, 1, 1, T>(a, G, Hb, Gb, st);
  if constexpr (sizeof(T) == 4) {
    if (L <= 128) return launch_xpass_adj_t<64, 2, 1, T>(a, G, Hb, Gb, st);
    if (L <= 192) return launch_xpass_adj_t<64, 3, 1, T>(a, G, Hb, Gb, st);
    if (L <= 384) return launch_xpass_adj_t<128, 3, 1, T>(a, G, Hb, Gb, st);
    if (L <= 768) return launch_xpass_adj_t<256, 3, 1, T>(a, G, Hb, Gb, st);
    if (L <= 1536) return launch_xpass_adj_t<512, 3, 1, T>(a, G, Hb, Gb, st);
    if (L <= 3072) return launch_xpass_adj_t<1024, 3, 1, T>(a, G, Hb, Gb, st);
    if (L <= 6144) return launch_xpass_adj_t<1024, 6, 2, T>(a, G, Hb, Gb, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_xpass_adj(const XformArgs& a, const void* G, const void* Hbar, void* Gbar,
                            hipStream_t st, bool fp32) {
  return fp32 ? launch_xpass_adj_T<float>(a, G, Hbar, Gbar, st)
              : launch_xpass_adj_T<double>(a, G, Hbar, Gbar, st);
}

template <int NT>
static hipError_t launch_ke_row_adj_t(const XformArgs& a, const void* G, const void* ebar,
                                      void* Gb, hipStream_t st) {
  size_t lds = (size_t)a.L * sizeof(double2);
  allow_lds((const void*)ke_row_adj_kernel<2, 6, NT>, lds);
  hipLaunchKernelGGL((ke_row_adj_kernel<2, 6, NT>), dim3(a.M), dim3(NT), lds, st, a,
                     (const double2*)G, (const double2*)ebar, (double2*)Gb);
  return hipGetLastError();
}

hipError_t launch_ke_adjoint(const XformArgs& a, const void* X, void* G, void* Gbar,
                             const void* wvec, void* ebar, void* Xbar, hipStream_t st) {
  // e_bar_j: weighted DCT-III of the integration weights (one "pencil")
  XformArgs aw = a;
  aw.P = 1;
  aw.Pa = 1;
  aw.dim = 2;
  FieldList fw{};
  fw.nf = 1;
  fw.var[0] = 0;
  fw.src_S = 1;
  fw.wmode = 1;
  launch_zb(aw, fw, wvec, ebar, st);
  FieldList fl{};
  fl.nf = 2;
  fl.var[0] = 2;                   // u
  fl.var[1] = a.dim == 2 ? 3 : 4;  // w
  launch_zb(a, fl, X, G, st);
  hipError_t e;
  switch (x_threads(a.L)) {
    case 64: e = launch_ke_row_adj_t<64>(a, G, ebar, Gbar, st); break;
    case 128: e = launch_ke_row_adj_t<128>(a, G, ebar, Gbar, st); break;
    case 256: e = launch_ke_row_adj_t<256>(a, G, ebar, Gbar, st); break;
    case 512: e = launch_ke_row_adj_t<512>(a, G, ebar, Gbar, st); break;
    case 1024: e = launch_ke_row_adj_t<1024>(a, G, ebar, Gbar, st); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  e = hipMemsetAsync(Xbar, 0, (size_t)a.P * a.S * a.N * sizeof(double2), st);
  if (e != hipSuccess) return e;
  AccList al{};
  al.nt = 2;
  al.target[0] = 2;
  al.nsrc[0] = 1;
  al.src[0][0] = 0;
  al.target[1] = a.dim == 2 ? 3 : 4;
  al.nsrc[1] = 1;
  al.src[1][0] = 1;
  return launch_zadj(a, al, Gbar, Xbar, st);
}

hipError_t launch_initial_state_adjoint(const XformArgs& a1, const void* Xbar, double* gbar,
                                        void* work, hipStream_t st) {
  double2* C = (double2*)work;              // [P][1][N]
  double2* H1 = C + (size_t)a1.P * a1.N;    // [N][P]
  const int vb = 1, vbz = a1.dim == 2 ? 4 : 5;
  hipLaunchKernelGGL(ic_adj_coef_kernel, dim3((a1.P + 63) / 64), dim3(64), 0, st, a1,
                     (const double2*)Xbar, C, vb, vbz);
  FieldList fl{};
  fl.nf = 1;
  fl.var[0] = 0;
  fl.src_S = 1;
  fl.wmode = 1;
  launch_zb(a1, fl, C, H1, st);
  allow_lds((const void*)ic_adj_x_kernel<8>, (size_t)a1.Nx * sizeof(double2));
  hipLaunchKernelGGL((ic_adj_x_kernel<8>), dim3(a1.N), dim3(256), (size_t)a1.Nx * sizeof(double2),
                     st, a1, (const double2*)H1, gbar);
  return hipGetLastError();
}

}  // namespace stau
