// Pencil solve of the step by reduction to tridiagonal systems.
//
// Without a non-constant coefficient the first-order tau system of a pencil
// splits exactly (same unknowns, same equations, same boundary rows) into
// second-order systems of the form
//   al C q - kap D qz = f,   C qz - D q = 0   (U-rows 0 .. N - 2)
// with C the T-to-U conversion and D the derivative:
//   * b with al = a0 + kappa k^2 and its Dirichlet values;
//   * in 3-D the horizontal velocity normal to (kx, ky), with al = a0 + nu k^2;
//   * the vorticity eta = uz' + k w of the velocity along (kx, ky), U = i u_L
//     (uz' = i (u_L)_z, w and p as they are):  with phi the T coefficients whose
//     C gives the right-hand side of the U rows and g that of the w rows plus
//     the buoyancy C b,
//       al C eta - nu D zeta = k g + D phi,  C zeta - D eta = 0,
//     the pressure from s = phi + nu zeta = a0 U - k p;
//   * the stream function psi with U = -psi_z, w = k psi (continuity):
//       k^2 C psi - D psi_z = C eta,  C psi_z - D psi = 0.
// b, the normal velocity and psi have boundary values; eta is the response
// with zero wall values plus t times the response to unit wall values, t from
// the walls' U = 0.  (k = 0: psi's net flux is free, s_0 = a0 U_0 instead, and
// p takes the gauge p(1) = 0.)
//
// C and D couple degrees of one parity, so each second-order system is two
// chains in q, stride 2 in the degree.  With x = al / kap, B_m = x / (8 (m + 1))
// (0 at m = N - 1), A_m = B_{m-2}, fh_m = f_m / (4 kap (m + 1)) and the fluxes
// F_m = qz_{m+1} / 2 (F_{-1} = qz_0) the rows are
//   F_m = B_m (q_m - q_{m+2}) - fh_m,   F_{m-2} = F_m + 2 m q_m
// (m = 0: F_0 = B_0 (2 q_0 - q_2) - fh_0).  Eliminated from the highest degree
// downwards,
//   F_m = b_m q_m - S_m,   b_m = B_m ratio_{m+2},   u_m = 2 m + b_m,
//   ratio_m = u_m / (A_m + u_m),   S_{m-2} = (1 - ratio_m) S_m + ratio_m fh_{m-2},
// and upwards q_m = (F_{m-2} + S_m) / u_m, F_m = (b_m F_{m-2} - 2 m S_m) / u_m:
// every coefficient is a ratio of sums of positive terms (S an average of fh),
// so nothing cancels in the factors, and q and qz come out together, each
// accurate in its own scale.  The boundary row sum q = G fixes the first flux.
// Against 80-bit solutions over k <= 6400, dt >= 1e-5 the worst field's error is
//   random right-hand sides (N <= 128):   6e-16 in the median, 2.3e-13 at most
//     (a dense LU with partial pivoting: 7e-15 and 1e-10);
//   a step's (a0 M X of an admissible state outweighs the rest, N <= 64):
//     1e-13 in the median, 5e-10 at most (LU 2e-13 and 5e-10), for both in bz,
//     uz and p; b, U, w and wz stay within 4e-15 (LU 2.5e-11).
//
// Factor tables per distinct wavenumber modulus k (a 3-D domain of a square
// box has one for up to eight pencils), kTauArrays arrays of N doubles: ratio and
// 1 / u of b, of eta (and the normal velocity) and of psi, then the unit-wall
// responses eta, psi, U and p; and kTauScal scalars (TauScal).
#include <algorithm>

#include "pencil.h"

namespace stau {

namespace {

// table arrays: two per system (b, eta, psi), then the unit-wall responses
enum TauArray { kRatio = 0, kUi = 1, kHe = 6, kHp, kHu, kHpr };
// scalars: k; per system the sums of the homogeneous q (first flux 1) over the
// even and odd degrees >= 1 and b_0; the unit-wall sums of U; the mean pencil's
// denominator of t
enum TauScal { kScK = 0, kScSys = 1, kScU = 10, kScMean = 12 };

__device__ __forceinline__ double cfac(int n) { return n == 0 ? 1.0 : 0.5; }

// first flux of a chain of parity c from its boundary sum G, the sum sig of the
// particular q over degrees >= 1 (first flux 0), S_0 and the scalars h = (sums of
// the homogeneous q, b_0) of the system
__device__ __forceinline__ double first_flux(int c, double G, double sig, double S0, const double* h) {
  if (c == 0) {
    const double b2 = 2.0 * h[2];
    return (b2 * (G - sig) - S0) / fma(b2, h[0], 1.0);
  }
  return (G - sig) / h[1];
}

}  // namespace

// ---------------------------------------------------------------------------
// Tables of one operator a0 M~ + L~, KB wavenumbers per block, all in LDS; the
// tables leave as one contiguous copy.  Bound by the elimination's chain of N / 2
// dependent divisions (six lanes per wavenumber: system, parity).  What is not a
// recurrence runs over all threads by (wavenumber, degree), and the two
// recurrences of the unit-wall response of psi have products and sums only
// (64x64x64: 46 -> 23 us against six lanes doing everything; the banded LU
// factors of the same operator 1520 us).
// ---------------------------------------------------------------------------
constexpr int kTauWork = 4;  // working arrays beside the tables: b and homogeneous fluxes per system, nu zeta
constexpr int kTauThreads = 256;
__global__ void __launch_bounds__(kTauThreads) tau_factor_kernel(int N, int lgN, int nk, int KB, double a0,
                                                                 double kappa, double nu,
                                                                 const double* __restrict__ kmod,
                                                                 double* __restrict__ tab, double* __restrict__ scal,
                                                                 [[maybe_unused]] unsigned* check) {
  extern __shared__ double lds[];
  const int tid = threadIdx.x;
  const int k0 = blockIdx.x * KB, nkb = min(KB, nk - k0);
  const int KS = (kTauArrays + kTauWork) * N + kTauScal + 1;  // stride per wavenumber
  const int n = N / 2;
  double* inv = lds + (size_t)KB * KS;                        // 1 / m
  auto T_of = [&](int kb) {
    STAU_BOUND(check, kb >= 0 && kb < KB && k0 + kb < nk, kChkTau);
    return lds + (size_t)kb * KS;
  };
  auto sc_of = [&](int kb) { return lds + (size_t)kb * KS + (kTauArrays + kTauWork) * N; };
  // f(kb, m) for every wavenumber and degree
  auto each = [&](auto&& f) {
    for (int idx = tid; idx < nkb << lgN; idx += kTauThreads) {
      STAU_BOUND(check, idx >> lgN < nkb && (1 << lgN) == N, kChkTau);
      f(idx >> lgN, idx & (N - 1));
    }
  };
  for (int m = tid + 1; m <= N; m += kTauThreads) inv[m] = 1.0 / (double)m;
  if (tid < nkb) sc_of(tid)[kScK] = kmod[k0 + tid];
  __syncthreads();
  const int kb6 = tid / 6, sys6 = (tid % 6) >> 1, par6 = tid & 1;
  if (kb6 < nkb) {
    double* T = T_of(kb6);
    const double k = sc_of(kb6)[kScK], k2 = k * k;
    const double x = sys6 == 0 ? (a0 + kappa * k2) / kappa : (sys6 == 1 ? (a0 + nu * k2) / nu : k2);
    const double x8 = 0.125 * x;
    double *rat = T + (2 * sys6 + kRatio) * N, *u_ = T + (2 * sys6 + kUi) * N, *ph = T + (kTauArrays + sys6) * N;
    double r2 = 1.0;  // ratio_{m+2}
    for (int j = n - 1; j >= 0; --j) {
      const int m = 2 * j + par6;
      const double b = m + 1 <= N - 1 ? x8 * inv[m + 1] * r2 : 0.0;
      if (m == 0) {
        rat[0] = 0.0;
        ph[0] = b;
        break;
      }
      const double u = 2.0 * m + b;
      const double A = m >= 2 ? x8 * inv[m - 1] : 0.0;
      u_[m] = u;
      ph[m] = b;
      r2 = u / (A + u);
      rat[m] = r2;
    }
  }
  __syncthreads();
  each([&](int kb, int m) {
    double* T = T_of(kb);
#pragma unroll
    for (int sys = 0; sys < 3; ++sys) {
      double *ui = T + (2 * sys + kUi) * N, *ph = T + (kTauArrays + sys) * N;
      if (m == 0) {
        sc_of(kb)[kScSys + 3 * sys + 2] = ph[0];
        ui[0] = 0.0;
        ph[0] = 1.0;
      } else {
        const double v = 1.0 / ui[m];
        ui[m] = v;
        ph[m] *= v;
      }
    }
  });
  __syncthreads();
  // homogeneous solutions with first flux 1
  if (kb6 < nkb) {
    double* T = T_of(kb6);
    double *ui = T + (2 * sys6 + kUi) * N, *ph = T + (kTauArrays + sys6) * N;
    double v = 1.0, H = 0.0;
    for (int j = par6 == 0 ? 1 : 0; j < n; ++j) {
      const int m = 2 * j + par6;
      H = fma(v, ui[m], H);
      v *= ph[m];
      ph[m] = v;
    }
    sc_of(kb6)[kScSys + 3 * sys6 + par6] = H;
  }
  __syncthreads();
  // eta with boundary sum 1, and nu zeta
  each([&](int kb, int m) {
    double* T = T_of(kb);
    const double* hn = sc_of(kb) + kScSys + 3;
    const double *uin = T + (2 + kUi) * N, *phn = T + (kTauArrays + 1) * N;
    double *he = T + kHe * N, *hs = T + (kTauArrays + 3) * N;
    const double st = first_flux(m & 1, 1.0, 0.0, 0.0, hn);
    he[m] = m == 0 ? 1.0 - hn[0] * st : (m >= 2 ? st * phn[m - 2] : st) * uin[m];
    if (m + 1 < N) hs[m + 1] = 2.0 * nu * (st * phn[m]);
    if (m == 1) hs[0] = nu * st;
  });
  __syncthreads();
  // psi with boundary sum 0: the sources of S in hp, b and the factors of S in the
  // working arrays of b and eta
  each([&](int kb, int m) {
    double* T = T_of(kb);
    const double k = sc_of(kb)[kScK], k2 = k * k, al = a0 + nu * k2;
    const double *he = T + kHe * N, *hs = T + (kTauArrays + 3) * N;
    const double *rp = T + (4 + kRatio) * N, *uip = T + (4 + kUi) * N;
    const double r2 = m + 2 < N ? rp[m + 2] : 1.0;
    const double b = m + 1 <= N - 1 ? 0.125 * k2 * inv[m + 1] * r2 : 0.0;
    // C eta: the differences of eta cancel where al dominates; there al C eta =
    // nu D zeta
    double ce = 0.0;
    if (m <= N - 2) {
      const double d = (double)(m + 1);
      ce = al > 4.0 * nu * d * d ? 2.0 * d * hs[m + 1] / al : cfac(m) * he[m] - (m + 2 < N ? 0.5 * he[m + 2] : 0.0);
    }
    T[kHp * N + m] = r2 * (0.25 * ce * inv[m + 1]);
    T[kTauArrays * N + m] = b;
    T[(kTauArrays + 1) * N + m] = b * (m + 2 < N ? uip[m + 2] : 0.0);
  });
  __syncthreads();
  const int kb2 = tid >> 1, e2 = tid & 1;  // e: parity of eta, psi
  if (kb2 < nkb) {
    double *T = T_of(kb2), *sc = sc_of(kb2);
    const double *uip = T + (4 + kUi) * N, *bp = T + kTauArrays * N, *alp = T + (kTauArrays + 1) * N;
    double *hp = T + kHp * N, *hu = T + kHu * N;
    double v = 0.0;
    for (int j = n - 1; j >= 0; --j) {
      const int m = 2 * j + e2;
      v = fma(alp[m], v, hp[m]);
      hp[m] = v;
    }
    double sig = 0.0;
    v = 0.0;
    for (int j = 0; j < n; ++j) {
      const int m = 2 * j + e2;
      const double ui = uip[m], S = hp[m];
      sig = fma(v + S, ui, sig);
      v = fma(bp[m], v, -2.0 * m * S) * ui;
      if (m + 1 < N) hu[m + 1] = v;
    }
    // (the sums of U's place holds the first fluxes, kScMean's and the unused slot
    // behind the scalars the sums of the particular psi until they are used)
    sc[kScU + e2] = first_flux(e2, 0.0, sig, hp[e2 ? 1 : 0], sc + kScSys + 6);
    sc[kScMean + e2] = sig;
  }
  __syncthreads();
  // psi, then U = -psi_z, each in place
  each([&](int kb, int m) {
    double* T = T_of(kb);
    const double* sc = sc_of(kb);
    const double sp = sc[kScU + (m & 1)];
    const double fl = m >= 2 ? T[kHu * N + m - 1] + sp * T[(kTauArrays + 2) * N + m - 2] : sp;
    T[kHp * N + m] = m == 0 ? -sc[kScMean] - sc[kScSys + 6] * sp : (fl + T[kHp * N + m]) * T[(4 + kUi) * N + m];
  });
  __syncthreads();
  each([&](int kb, int m) {
    double* T = T_of(kb);
    const double* sc = sc_of(kb);
    double* hu = T + kHu * N;
    if (m + 1 < N) hu[m + 1] = -2.0 * (hu[m + 1] + sc[kScU + (m & 1)] * T[(kTauArrays + 2) * N + m]);
    if (m == 1) hu[0] = -sc[kScU + 1];
  });
  __syncthreads();
  if (kb2 < nkb) {
    double *T = T_of(kb2), *sc = sc_of(kb2);
    const double *hu = T + kHu * N, *hs = T + (kTauArrays + 3) * N;
    double sum = 0.0;
    for (int m = 1 - e2; m < N; m += 2) sum += hu[m];
    // t of the mean pencil: s_0 = a0 U_0 once sum U = 0
    if (e2 == 1) sc[kScMean] = hs[0] - a0 * (hu[0] - sum);
    sc[kScU + e2] = sum;
  }
  // p: D p = -a0 C w - nu k C eta where the degree exceeds k / 2, else k p = a0 U - s
  each([&](int kb, int m) {
    double* T = T_of(kb);
    const double k = sc_of(kb)[kScK];
    const double *he = T + kHe * N, *hp = T + kHp * N;
    double p = 0.0;
    if (m >= 1 && k < 2.0 * m) {
      const int l = m - 1;
      double ce = cfac(l) * he[l], cp = cfac(l) * hp[l];
      if (l + 2 < N) {
        ce -= 0.5 * he[l + 2];
        cp -= 0.5 * hp[l + 2];
      }
      p = -0.5 * k * (a0 * cp + nu * ce) * inv[m];
    } else if (k > 0.0) {
      p = (a0 * T[kHu * N + m] - T[(kTauArrays + 3) * N + m]) / k;
    }
    T[kHpr * N + m] = p;
  });
  __syncthreads();
  const int per = kTauArrays * N;
  for (int kb = 0; kb < nkb; ++kb) {
    const double* T = T_of(kb);
    for (int i = tid; i < per; i += kTauThreads) tab[(size_t)(k0 + kb) * per + i] = T[i];
    if (tid < kTauScal) scal[(size_t)(k0 + kb) * kTauScal + tid] = sc_of(kb)[tid];
  }
}

// ---------------------------------------------------------------------------
// Chains.  The N / 2 degrees m = 2 j + c of a parity c and real part of an array
// are E consecutive j on each of L lanes of a row of 16 (L a power of two): both
// recurrences run on registers, over the lane's own elements, then over the
// lanes by a scan of (offset, factor) pairs, then over its elements again
// from the value that enters it.  In LDS the four chains (parity, part) of an
// array follow each other, lane blocks one double apart, so that the L lanes
// read distinct banks.
// ---------------------------------------------------------------------------
namespace {

// values of the lane d further up / down the row, of the row's lanes with one
// bit of the lane index flipped
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int D>
__device__ __forceinline__ double from_up(double v) { return dpp<0x100 | D>(v); }
template <int D>
__device__ __forceinline__ double from_down(double v) { return dpp<0x110 | D>(v); }

// sum over the L lanes of a chain, on all of them
__device__ __forceinline__ double chain_sum(double v, int L) {
  if (L > 1) v += dpp<0xB1>(v);   // lanes 1 apart
  if (L > 2) v += dpp<0x4E>(v);   // pairs
  if (L > 4) v += dpp<0x141>(v);  // quads (mirrored halves of eight)
  if (L > 8) v += dpp<0x140>(v);  // halves of the row
  return v;
}

// v_j = al_j v_{j+1} + s_j (UP) or v_j = al_j v_{j-1} + s_j: the value entering
// this lane's block from its block's (offset v, factor pi); pi becomes the factor from
// the chain's start to this block
template <bool UP>
__device__ __forceinline__ double chain_enter(double v, double& pi, int g, int L) {
  auto level = [&](auto d) {
    constexpr int D = decltype(d)::value;
    if (D < L) {
      const double v2 = UP ? from_up<D>(v) : from_down<D>(v), p2 = UP ? from_up<D>(pi) : from_down<D>(pi);
      if (UP ? g + D < L : g >= D) {
        v = fma(pi, v2, v);
        pi *= p2;
      }
    }
  };
  level(std::integral_constant<int, 1>{});
  level(std::integral_constant<int, 2>{});
  level(std::integral_constant<int, 4>{});
  level(std::integral_constant<int, 8>{});
  const double in = UP ? from_up<1>(v) : from_down<1>(v), pin = UP ? from_up<1>(pi) : from_down<1>(pi);
  const bool edge = UP ? g + 1 >= L : g == 0;
  pi = edge ? 1.0 : pin;
  return edge ? 0.0 : in;
}

// What a chain leaves beside q and its fluxes: first flux, sum of the fluxes
struct TauStart {
  double2 f[2], sum[2];
};

// One chain with boundary sum G: S (ratio_{m+2} fh_m) becomes q, F the fluxes;
// bc = b, ui = 1 / u, h the system's scalars
template <int E>
__device__ __forceinline__ void tau_chain(double* S, double* F, const double* bc, const double* ui, const double* h,
                                          double G, int g, int L, int c, int part, TauStart* out) {
  const int o = g * (E + 1);
  double s[E], b[E], u[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    s[i] = S[o + i];
    b[i] = bc[o + i];
    u[i] = ui[o + i];
  }
  const double un = g + 1 < L ? ui[o + E + 1] : 0.0;  // of the next lane's first degree
  {
    double v = 0.0, pi = 1.0;
#pragma unroll
    for (int i = E - 1; i >= 0; --i) {
      const double al = b[i] * (i + 1 < E ? u[i + 1 < E ? i + 1 : i] : un);
      v = fma(al, v, s[i]);
      pi *= al;
    }
    v = chain_enter<true>(v, pi, g, L);
#pragma unroll
    for (int i = E - 1; i >= 0; --i) {
      v = fma(b[i] * (i + 1 < E ? u[i + 1 < E ? i + 1 : i] : un), v, s[i]);
      s[i] = v;
    }
  }
  // upwards: be = b / u (1 at m = 0, whose flux is the first one)
  const bool bottom = g == 0 && c == 0;
  const int m0 = 2 * g * E + c;
  const double S0 = chain_sum(g == 0 ? s[0] : 0.0, L);
  double v = 0.0, pi = 1.0, sig = 0.0, hh = 0.0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const double w = u[i] * s[i];
    b[i] = i == 0 && bottom ? 1.0 : b[i] * u[i];
    sig += fma(v, u[i], w);
    hh = fma(pi, u[i], hh);
    v = fma(b[i], v, -(double)(2 * (m0 + 2 * i)) * w);
    pi *= b[i];
  }
  v = chain_enter<false>(v, pi, g, L);
  sig = chain_sum(fma(hh, v, sig), L);
  const double st = first_flux(c, G, sig, S0, h);
  v = fma(pi, st, v);
  double sum = 0.0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const double q = (v + s[i]) * u[i];
    v = fma(b[i], v, -(double)(2 * (m0 + 2 * i)) * (u[i] * s[i]));
    sum += v;
    S[o + i] = q;
    F[o + i] = v;
  }
  sum = chain_sum(sum, L);
  if (g == 0) {
    if (c == 0) S[0] = G - sig - h[0] * st;
    ((double*)&out->f[c])[part] = st;
    ((double*)&out->sum[c])[part] = sum;
  }
}

__device__ __forceinline__ double2 operator*(double s, double2 v) { return make_double2(s * v.x, s * v.y); }
__device__ __forceinline__ double2 operator+(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 operator-(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

}  // namespace

// ---------------------------------------------------------------------------
// The solve: NP consecutive pencils per block, one (pencil, degree) per thread:
// it reads its rows of the right-hand sides and its table entries at the start
// and writes its nine (2-D: seven) state entries, every access contiguous over
// the degrees; neighbouring degrees' values come from LDS.  The chains of the
// independent systems run on different wavefronts.  LDS per pencil: NA arrays
// (b and its fluxes, then psi's; eta's; phi; g; 3-D: the normal velocity's)
// and four coefficient arrays (b, 1 / u of b, then of psi; of eta).
// Bound by the memory at the large sizes (256x256x128: 297 us, 0.95 GB; one lane
// per chain 766, the banded sweeps 3195), by the three chains' latency at the
// small ones (1024x256: 16 us, 47, 124; 4096x64: 16, 26, 95; 64x32: 9.5, -, 20).
// ---------------------------------------------------------------------------
template <int DIM, int E>
__global__ void __launch_bounds__(E > 8 ? 512 : 256) tau_solve_kernel(PencilArgs a, TauFactors tf, double a0, int NP,
                                                                      int L, const double2* __restrict__ Bev,
                                                                      double2* __restrict__ X) {
  constexpr int NA = DIM == 3 ? 8 : 6, S = DIM == 3 ? 9 : 7, ne = DIM == 3 ? 4 : 3;
  constexpr int eW = ne - 1;
  // state layout (p, b, u, [v], w, bz, uz, [vz], wz)
  constexpr int vP = 0, vB = 1, vU = 2, vV = 3, vW = ne, vBz = ne + 1, vUz = ne + 2, vVz = ne + 3, vWz = S - 1;
  enum { AB = 0, AZ, AE, AX, AF, AG, AT, ATZ };
  extern __shared__ double lds[];
  const int N = a.desc.N, tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int PL = L * (E + 1);  // doubles per chain
  const int PS = (NA * 4 + 8) * PL;
  TauStart* starts = (TauStart*)lds;               // [NP][4]: b, the normal velocity, eta, psi
  double2* gauge = (double2*)(starts + 4 * NP);    // the mean pencil's sum of p over degrees >= 1
  double* base = (double*)(gauge + 1);
  // chain ch = 2 parity + part of an array; coefficients by parity
  auto chain_at = [&](int i, int which, int ch) {
    STAU_BOUND(a.check, i >= 0 && i < NP && which < NA && ch < 4, kChkTau);
    return base + (size_t)i * PS + (which * 4 + ch) * PL;
  };
  auto coef_at = [&](int i, int which, int c) {
    STAU_BOUND(a.check, i >= 0 && i < NP && which < 4 && c < 2, kChkTau);
    return base + (size_t)i * PS + (NA * 4 + which * 2 + c) * PL;
  };
  // place of degree m in its chain
  auto pos = [&](int m) {
    const int o = (m >> 1) + (m >> 1) / E;
    STAU_BOUND(a.check, m >= 0 && m < N && o < PL, kChkTau);
    return o;
  };

  // this thread's pencil and degree
  const int i = tid / N, m = tid - i * N, p = (int)blockIdx.x * NP + i;
  const bool mine = i < NP && p < a.P;
  const int slot = mine ? tf.slot[p] : -1;
  const bool on = slot >= 0;
  STAU_BOUND(a.check, slot < tf.nk, kChkTau);
  const double* T = tf.tab + (size_t)(on ? slot : 0) * (kTauArrays * N) + m;
  const double* sc = tf.scal + (size_t)(on ? slot : 0) * kTauScal;
  const double2 zero = make_double2(0.0, 0.0);
  const double inv1 = 1.0 / (double)(m + 1), invm = m ? 1.0 / (double)m : 0.0;
  double k = 0.0, cx = 1.0, cy = 0.0, r2[3], ui[3], he = 0.0, hp = 0.0, hu = 0.0, hpr = 0.0;
  double2 fw = zero;
  auto get = [&](int which, int l) {
    const double* q = chain_at(i, which, 2 * (l & 1)) + pos(l);
    return make_double2(q[0], q[PL]);
  };
  auto put = [&](int which, double2 v) {
    double* q = chain_at(i, which, 2 * (m & 1)) + pos(m);
    q[0] = v.x;
    q[PL] = v.y;
  };
  // b_m and 1 / u_m of system sys into the coefficient arrays w, w + 1
  auto coefs = [&](int sys, double x, int w) {
    coef_at(i, w, m & 1)[pos(m)] = m + 1 < N ? 0.125 * x * inv1 * r2[sys] : 0.0;
    coef_at(i, w + 1, m & 1)[pos(m)] = ui[sys];
  };

  // ---- right-hand sides of b, the normal velocity and phi ----
  if (on) {
    const bool row = m <= N - 2;
    const double2* B = Bev + (size_t)p * ne * N + m;
    const double2 fb = row ? B[0] : zero, f1 = row ? B[N] : zero, f2 = DIM == 3 && row ? B[2 * N] : zero;
    fw = row ? B[eW * N] : zero;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      r2[q] = m + 2 < N ? T[(2 * q + kRatio) * N + 2] : 1.0;
      ui[q] = T[(2 * q + kUi) * N];
    }
    he = T[kHe * N];
    hp = T[kHp * N];
    hu = T[kHu * N];
    hpr = T[kHpr * N];
    k = sc[kScK];
    if (DIM == 3 && k != 0.0) {
      const int iy = p / a.Px, ix = p - iy * a.Px;
      const int ky = iy < (a.Ny + 1) / 2 ? iy : iy - a.Ny;
      cx = a.two_pi_over_Lx * (double)ix / k;
      cy = a.two_pi_over_Ly * (double)ky / k;
    }
    const double k2 = k * k;
    coefs(0, (a0 + a.kappa * k2) / a.kappa, 0);
    coefs(1, (a0 + a.nu * k2) / a.nu, 2);
    put(AB, (0.25 * inv1 * r2[0] / a.kappa) * fb);
    double2 fu = f1;
    if (DIM == 3) {
      put(AT, (0.25 * inv1 * r2[1] / a.nu) * (cx * f2 - cy * f1));
      fu = cx * f1 + cy * f2;
    }
    // U = i u_L: its row is i times that of u_L; phi_m = 2 row_m + phi_{m+2}
    put(AF, (m ? 2.0 : 1.0) * make_double2(-fu.y, fu.x));
  }
  __syncthreads();

  // this lane's chain
  const int ch = lane / L, g = lane - ch * L, li = ch >> 2, c = (ch >> 1) & 1, part = ch & 1;
  const int lp = (int)blockIdx.x * NP + li;
  const int lslot = li < NP && lp < a.P ? tf.slot[lp] : -1;
  const double* lsc = tf.scal + (size_t)(lslot >= 0 ? lslot : 0) * kTauScal;
  auto chain = [&](int s, int f, int w, int sys, int which, double G) {
    // (its degrees, and the next lane's first where there is one)
    STAU_BOUND(a.check, g >= 0 && g < L && L * E == N / 2 && g * (E + 1) + E <= PL && lslot < tf.nk, kChkTau);
    tau_chain<E>(chain_at(li, s, ch & 3), chain_at(li, f, ch & 3), coef_at(li, w, c), coef_at(li, w + 1, c),
                 lsc + kScSys + 3 * sys, G, g, L, c, part, starts + li * 4 + which);
  };
  if (lslot >= 0) {
    if (wv == 0) {
      const bool mean = lsc[kScK] == 0.0 && part == 0;
      chain(AB, AZ, 0, 0, 0, mean ? 0.5 * (a.b_top + (c ? -a.b_bottom : a.b_bottom)) : 0.0);
    }
    if (DIM == 3 && wv == 1) chain(AT, ATZ, 2, 1, 1, 0.0);
    if (wv == 2) {
      double* f = chain_at(li, AF, ch & 3) + g * (E + 1);
      double s[E], v = 0.0, pi = 1.0;
#pragma unroll
      for (int q = E - 1; q >= 0; --q) {
        s[q] = f[q];
        v += s[q];
      }
      // (the factor 1 / 2 of m = 0 reaches no other degree)
      v = chain_enter<true>(v, pi, g, L);
#pragma unroll
      for (int q = E - 1; q >= 0; --q) {
        v = q == 0 && g == 0 && c == 0 ? fma(0.5, v, s[q]) : v + s[q];
        f[q] = v;
      }
    }
  }
  __syncthreads();

  // ---- b and b_z leave; g = row of w + buoyancy C b; right-hand side of eta ----
  double2 gw = zero, fh = zero;  // g_m, f_m / (4 nu (m + 1)) of eta
  const double k2 = k * k, al = a0 + a.nu * k2;
  double2* Xp = X + (size_t)p * S * N + m;
  if (on) {
    const double2 b = get(AB, m);
    Xp[vB * N] = b;
    Xp[vBz * N] = m ? 2.0 * get(AZ, m - 1) : starts[i * 4].f[1];
    if (m <= N - 2) {
      double2 cb = cfac(m) * b;
      if (m + 2 < N) cb = cb - 0.5 * get(AB, m + 2);
      gw = fw + a.buoyancy * cb;
      // f_m = k g_m + 2 (m + 1) phi_{m+1}
      fh = (1.0 / a.nu) * (0.25 * k * inv1 * gw + 0.5 * get(AF, m + 1));
    }
    put(AG, gw);
    put(AE, r2[1] * fh);
  }
  __syncthreads();

  // ---- eta with zero wall values; the mean pencil's gauge sum ----
  if (wv == 0 && lslot >= 0) chain(AE, AX, 2, 1, 2, 0.0);
  if (wv == 1 && blockIdx.x == 0) {  // (the mean pencil is the first)
    double2 sum = zero;
    for (int l = lane + 1; l < N; l += kWave) {
      const double* q = chain_at(0, AG, 2 * ((l - 1) & 1)) + pos(l - 1);
      sum = sum + (0.5 / (double)l) * make_double2(q[0], q[PL]);
    }
#pragma unroll
    for (int d = 32; d; d >>= 1) {
      sum.x += __shfl_xor(sum.x, d);
      sum.y += __shfl_xor(sum.y, d);
    }
    if (lane == 0) *gauge = sum;
  }
  __syncthreads();

  // ---- right-hand side of psi ----
  if (on) {
    double2 ce = zero;
    if (m <= N - 2) {
      // C eta, from al C eta = f + nu D zeta where the differences of eta cancel
      const double d = (double)(m + 1);
      if (al > 4.0 * a.nu * d * d) {
        ce = (4.0 * a.nu * d / al) * (fh + get(AX, m));
      } else {
        ce = cfac(m) * get(AE, m);
        if (m + 2 < N) ce = ce - 0.5 * get(AE, m + 2);
      }
    }
    put(AB, (0.25 * r2[2] * inv1) * ce);
    coefs(2, k2, 0);
  }
  __syncthreads();

  // ---- psi ----
  if (wv == 0 && lslot >= 0) chain(AB, AZ, 0, 2, 3, 0.0);
  __syncthreads();

  // ---- velocity and pressure ----
  if (!mine) return;
  if (!on) {
#pragma unroll
    for (int v = 0; v < S; ++v) Xp[v * N] = zero;
    return;
  }
  // wall vorticity t of either class from sum U = 0; U0: the mean pencil's free
  // constant of U
  const bool mean = k == 0.0;
  const TauStart &se = starts[i * 4 + 2], &sp = starts[i * 4 + 3];
  const double2 su0 = -2.0 * sp.sum[0], su1 = -2.0 * sp.sum[1] - sp.f[1];
  double2 t0 = (-1.0 / sc[kScU]) * su0, t1, U0 = zero;
  if (mean) {  // s_0 = a0 U_0 with sum U = 0
    t1 = (-1.0 / sc[kScMean]) * (get(AF, 0) + a.nu * se.f[1] + a0 * (sp.f[1] + su1));
    U0 = -1.0 * su1 - sc[kScU + 1] * t1;
  } else {
    t1 = (-1.0 / sc[kScU + 1]) * su1;
  }
  const double2 te = m & 1 ? t1 : t0, to = m & 1 ? t0 : t1;  // of the parity of m, of the other
  const double2 psi = get(AB, m), eta = get(AE, m);
  const double2 Up = m ? -2.0 * get(AZ, m - 1) : -1.0 * sp.f[1];
  double2 U = Up + hu * to;
  if (m == 0) U = U + U0;
  const double2 w = k * (psi + hp * te), uz = eta + he * te - k * w;
  // pressure: D p from the w rows where the degree exceeds k / 2, else from s
  double2 pr = hpr * to;
  if (m >= 1 && k < 2.0 * m) {
    const int l = m - 1;
    double2 ce = cfac(l) * get(AE, l), cp = cfac(l) * get(AB, l);
    if (l + 2 < N) {
      ce = ce - 0.5 * get(AE, l + 2);
      cp = cp - 0.5 * get(AB, l + 2);
    }
    pr = pr + 0.5 * invm * (get(AG, l) - (a0 * k) * cp - (a.nu * k) * ce);
  } else if (!mean) {
    const double2 s = get(AF, m) + a.nu * (m ? 2.0 * get(AX, m - 1) : se.f[1]);
    pr = pr + (1.0 / k) * (a0 * Up - s);
  } else {  // m = 0: gauge p(1) = 0 of the mean pencil
    pr = -1.0 * *gauge;
  }
  Xp[vP * N] = pr;
  Xp[vW * N] = w;
  Xp[vWz * N] = (-k) * U;
  // u_L = -i U
  const double2 ul = make_double2(U.y, -U.x), uzl = make_double2(uz.y, -uz.x);
  if (DIM == 3) {
    const double2 T0 = get(AT, m), Tz = m ? 2.0 * get(ATZ, m - 1) : starts[i * 4 + 1].f[1];
    Xp[vU * N] = cx * ul - cy * T0;
    Xp[vV * N] = cy * ul + cx * T0;
    Xp[vUz * N] = cx * uzl - cy * Tz;
    Xp[vVz * N] = cy * uzl + cx * Tz;
  } else {
    Xp[vU * N] = ul;
    Xp[vUz * N] = uzl;
  }
}

// ---------------------------------------------------------------------------
// Launches
// ---------------------------------------------------------------------------
static void allow_lds(const void* fn, size_t bytes) {
  if (bytes > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_tau_factor(const PencilArgs& a, double a0, const TauFactors& tf, hipStream_t st) {
  const int N = a.desc.N;
  // up to eight wavenumbers per block in half a compute unit's LDS, fewer while
  // that leaves units without a block
  const size_t per = (size_t)((kTauArrays + kTauWork) * N + kTauScal + 1) * sizeof(double);
  int KB = (int)std::max<size_t>(1, std::min<size_t>(8, (size_t)(72 * 1024) / per));
  while (KB > 1 && (tf.nk + KB - 1) / KB < tf.cus) --KB;
  const size_t lds = KB * per + (size_t)(N + 1) * sizeof(double);
  int lgN = 0;
  while ((1 << lgN) < N) ++lgN;
  allow_lds((const void*)tau_factor_kernel, lds);
  hipLaunchKernelGGL(tau_factor_kernel, dim3((tf.nk + KB - 1) / KB), dim3(kTauThreads), lds, st, N, lgN, tf.nk, KB, a0,
                     a.kappa, a.nu, tf.k, tf.tab, tf.scal, a.check);
  return hipGetLastError();
}

template <int DIM, int E>
static hipError_t launch_tau_solve_t(const PencilArgs& a, const TauFactors& tf, double a0, int NP, int L,
                                     const void* Bev, void* X, hipStream_t st) {
  constexpr int NA = DIM == 3 ? 8 : 6;
  const int threads = E > 8 ? 512 : 256;
  const size_t lds = NP * (4 * sizeof(TauStart) + (size_t)(NA * 4 + 8) * L * (E + 1) * sizeof(double)) + sizeof(double2);
  if (NP * a.desc.N > threads) return hipErrorInvalidValue;
  allow_lds((const void*)tau_solve_kernel<DIM, E>, lds);
  hipLaunchKernelGGL((tau_solve_kernel<DIM, E>), dim3((a.P + NP - 1) / NP), dim3(threads), lds, st, a, tf, a0, NP, L,
                     (const double2*)Bev, (double2*)X);
  return hipGetLastError();
}

hipError_t launch_tau_solve(const PencilArgs& a, const TauFactors& tf, double a0, const void* Bev, void* X,
                            hipStream_t st) {
  const int N = a.desc.N, n = N / 2;
  // pencils per block: one (pencil, degree) per thread of 256 (at most eight
  // pencils: 32 chains), fewer while that leaves compute units idle
  int NP = std::min(8, std::max(1, 256 / N));
  while (NP > 1 && (a.P + NP - 1) / NP < tf.cus) NP >>= 1;
  // the 4 NP chains of a block share a wavefront: lanes per chain, degrees per lane
  const int L = std::min(16 / NP, n), E = n / L;
#define STAU_TAU(EE)                                                                              \
  case EE:                                                                                        \
    return a.desc.dim == 3 ? launch_tau_solve_t<3, EE>(a, tf, a0, NP, L, Bev, X, st)              \
                           : launch_tau_solve_t<2, EE>(a, tf, a0, NP, L, Bev, X, st);
  switch (E) {
    STAU_TAU(1) STAU_TAU(2) STAU_TAU(4) STAU_TAU(8) STAU_TAU(16)
  }
#undef STAU_TAU
  return hipErrorInvalidValue;
}

}  // namespace stau
