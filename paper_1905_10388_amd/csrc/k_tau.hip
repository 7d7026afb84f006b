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
// Against 80-bit solutions of random right-hand sides over k <= 6400, dt >= 1e-5,
// N <= 128 the error per field is 6e-16 in the median and 2.3e-13 at most,
// where a dense LU with partial pivoting has 7e-15 and 1e-10.
//
// Factor tables per distinct wavenumber modulus k (a 3-D domain of a square
// box has one for up to eight pencils), kTauArrays arrays of N doubles: ratio,
// 1 / u and the homogeneous fluxes (first flux 1) of b, of eta (and the normal
// velocity) and of psi, then the unit-wall responses eta, psi, U and nu zeta;
// and kTauScal scalars (TauScal).
#include <algorithm>

#include "pencil.h"

namespace stau {

namespace {

// table arrays: three per system (b, eta, psi), then the unit-wall responses
enum TauArray { kRatio = 0, kUi = 1, kPh = 2, kHe = 9, kHp, kHu, kHs };
// scalars: k; per system the sums of the homogeneous q over the even and odd
// degrees >= 1 and b_0; the sums of psi's homogeneous fluxes; the unit-wall sums of U
enum TauScal { kScK = 0, kScSys = 1, kScPh = 10, kScU = 12 };

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
// Tables of one operator a0 M~ + L~.  One wavefront per block of KB
// wavenumbers: six lanes per wavenumber eliminate (system, parity), then two
// lanes form the unit-wall responses of the two parities, all in LDS; the
// tables leave as one contiguous copy.  A serial chain of N / 2 pairs of
// divisions bounds it.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kWave) tau_factor_kernel(int N, int nk, int KB, double a0, double kappa, double nu,
                                                           const double* __restrict__ kmod, double* __restrict__ tab,
                                                           double* __restrict__ scal) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x;
  const int k0 = blockIdx.x * KB, nkb = min(KB, nk - k0);
  const int KS = kTauArrays * N + kTauScal + 2;  // stride per wavenumber (staggers the banks)
  const int n = N / 2;
  {
    const int kb = lane / 6, sys = (lane % 6) >> 1, par = lane & 1;
    if (kb < nkb) {
      double* T = lds + (size_t)kb * KS;
      double* sc = T + kTauArrays * N;
      const double k = kmod[k0 + kb], k2 = k * k;
      const double x = sys == 0 ? (a0 + kappa * k2) / kappa : (sys == 1 ? (a0 + nu * k2) / nu : k2);
      const double x8 = 0.125 * x;
      double *rat = T + (3 * sys + kRatio) * N, *ui = T + (3 * sys + kUi) * N, *ph = T + (3 * sys + kPh) * N;
      double r2 = 1.0;  // ratio_{m+2}
      for (int j = n - 1; j >= 0; --j) {
        const int m = 2 * j + par;
        const double b = m + 1 <= N - 1 ? x8 / (double)(m + 1) * r2 : 0.0;
        if (m == 0) {
          rat[0] = ui[0] = 0.0;
          ph[0] = 1.0;
          sc[kScSys + 3 * sys + 2] = b;
          break;
        }
        const double u = 2.0 * m + b;
        const double A = m >= 2 ? x8 / (double)(m - 1) : 0.0;
        ui[m] = 1.0 / u;
        ph[m] = b;
        r2 = u / (A + u);
        rat[m] = r2;
      }
      double v = 1.0, H = 0.0, sum = par == 0 ? 1.0 : 0.0;
      for (int j = par == 0 ? 1 : 0; j < n; ++j) {
        const int m = 2 * j + par;
        H = fma(v, ui[m], H);
        v *= ph[m] * ui[m];
        ph[m] = v;
        sum += v;
      }
      sc[kScSys + 3 * sys + par] = H;
      if (sys == 2) sc[kScPh + par] = sum;
      if (sys == 0 && par == 0) sc[kScK] = k;
    }
  }
  __syncthreads();
  {
    const int kb = lane >> 1, e = lane & 1;  // e: parity of eta, psi
    if (kb < nkb) {
      double* T = lds + (size_t)kb * KS;
      double* sc = T + kTauArrays * N;
      const double k2 = sc[kScK] * sc[kScK], al = a0 + nu * k2;
      const double *uin = T + (3 + kUi) * N, *phn = T + (3 + kPh) * N;
      const double *rp = T + (6 + kRatio) * N, *uip = T + (6 + kUi) * N, *php = T + (6 + kPh) * N;
      double *he = T + kHe * N, *hp = T + kHp * N, *hu = T + kHu * N, *hs = T + kHs * N;
      // eta with boundary sum 1, and nu zeta
      const double* hn = sc + kScSys + 3;
      const double st = first_flux(e, 1.0, 0.0, 0.0, hn);
      if (e == 0)
        he[0] = 1.0 - hn[0] * st;
      else
        hs[0] = nu * st;
      double below = st;
      for (int j = 0; j < n; ++j) {
        const int m = 2 * j + e;
        if (m >= 1) he[m] = below * uin[m];
        below = st * phn[m];
        if (m + 1 < N) hs[m + 1] = 2.0 * nu * below;
      }
      // C eta: the differences of eta cancel where al dominates; there al C eta =
      // nu D zeta
      auto ceta = [&](int m) -> double {
        if (m > N - 2) return 0.0;
        const double d = (double)(m + 1);
        if (al > 4.0 * nu * d * d) return 2.0 * d * hs[m + 1] / al;
        return cfac(m) * he[m] - (m + 2 < N ? 0.5 * he[m + 2] : 0.0);
      };
      // psi with boundary sum 0: S in hp, the particular fluxes in hu
      const double x8 = 0.125 * k2;
      double v = 0.0;
      for (int j = n - 1; j >= 0; --j) {
        const int m = 2 * j + e;
        const double r2 = m + 2 < N ? rp[m + 2] : 1.0;
        const double b = m + 1 <= N - 1 ? x8 / (double)(m + 1) * r2 : 0.0;
        v = b * (m + 2 < N ? uip[m + 2] : 0.0) * v + r2 * (ceta(m) / (4.0 * (m + 1)));
        hp[m] = v;
      }
      double sig = 0.0, sphi = 0.0;
      v = 0.0;
      for (int j = 0; j < n; ++j) {
        const int m = 2 * j + e;
        const double r2 = m + 2 < N ? rp[m + 2] : 1.0;
        const double b = m + 1 <= N - 1 ? x8 / (double)(m + 1) * r2 : 0.0;
        sig += (v + hp[m]) * uip[m];
        v = (b * v - 2.0 * m * hp[m]) * uip[m];
        if (m + 1 < N) hu[m + 1] = v;
        sphi += v;
      }
      const double* hps = sc + kScSys + 6;
      const double sp = first_flux(e, 0.0, sig, hp[0], hps);
      sc[kScU + e] = -2.0 * (sphi + sp * sc[kScPh + e]) - (e == 1 ? sp : 0.0);
      double fl = sp;
      for (int j = 0; j < n; ++j) {
        const int m = 2 * j + e;
        hp[m] = m == 0 ? -sig - hps[0] * sp : (fl + hp[m]) * uip[m];
        if (m + 1 < N) {
          fl = hu[m + 1] + sp * php[m];
          hu[m + 1] = -2.0 * fl;
        }
      }
      if (e == 1) hu[0] = -sp;
    }
  }
  __syncthreads();
  const int per = kTauArrays * N;
  for (int kb = 0; kb < nkb; ++kb) {
    const double* T = lds + (size_t)kb * KS;
    for (int i = lane; i < per; i += kWave) tab[(size_t)(k0 + kb) * per + i] = T[i];
    if (lane < kTauScal) scal[(size_t)(k0 + kb) * kTauScal + lane] = T[per + lane];
  }
}

// ---------------------------------------------------------------------------
// Serial passes of one lane over the degrees m = 2 j + c of its parity c of one
// real part of complex arrays in LDS (pointers at that part; degree m at
// [2 m]).  n = N / 2 elements (a power of two), taken in chunks whose loads are
// issued one chunk ahead of the chain that consumes them: the chain is then
// one FMA per degree, not an LDS latency.
// ---------------------------------------------------------------------------
namespace {

constexpr int kTauCH = 8;

// load(j, buffer, slot) then step(j, buffer, slot) for j = n - 1 .. 0 (DOWN) or
// 0 .. n - 1
template <bool DOWN, typename LD, typename ST>
__device__ __forceinline__ void tau_pass(int n, LD&& load, ST&& step) {
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  auto at = [&](int q, int i) { return DOWN ? n - 1 - (q * kTauCH + i) : q * kTauCH + i; };
  if (n < kTauCH) {
    for (int i = 0; i < n; ++i) {
      load(at(0, i), B0{}, std::integral_constant<int, 0>{});
      step(at(0, i), B0{}, std::integral_constant<int, 0>{});
    }
    return;
  }
  const int nc = n / kTauCH;
  static_for<0, kTauCH>([&](auto i) { load(at(0, i), B0{}, i); });
  for (int q = 0; q < nc; q += 2) {
    if (q + 1 < nc) static_for<0, kTauCH>([&](auto i) { load(at(q + 1, i), B1{}, i); });
    static_for<0, kTauCH>([&](auto i) { step(at(q, i), B0{}, i); });
    if (q + 1 < nc) {
      if (q + 2 < nc) static_for<0, kTauCH>([&](auto i) { load(at(q + 2, i), B0{}, i); });
      static_for<0, kTauCH>([&](auto i) { step(at(q + 1, i), B1{}, i); });
    }
  }
}

// One chain: S holds ratio_{m+2} fh_m on entry and S_m on exit, F the particular
// fluxes (first flux 0); bc = b, ui = 1 / u by degree.  Returns the sum of the
// particular q over degrees >= 1, and the sum of F in *sumF.
__device__ __forceinline__ double tau_chain(double* S, double* F, const double* bc, const double* ui, int n, int c,
                                            double* sumF) {
  {
    double v = 0.0, up = 0.0;
    double sv[2][kTauCH], bv[2][kTauCH], uv[2][kTauCH];
    tau_pass<true>(
        n,
        [&](int j, auto b, auto i) {
          const int m = 2 * j + c;
          sv[b][i] = S[2 * m];
          bv[b][i] = bc[m];
          uv[b][i] = ui[m];
        },
        [&](int j, auto b, auto i) {
          v = fma(bv[b][i] * up, v, sv[b][i]);
          up = uv[b][i];
          S[2 * (2 * j + c)] = v;
        });
  }
  double v = 0.0, sig = 0.0, sf = 0.0;
  double sv[2][kTauCH], bv[2][kTauCH], uv[2][kTauCH];
  tau_pass<false>(
      n,
      [&](int j, auto b, auto i) {
        const int m = 2 * j + c;
        sv[b][i] = S[2 * m];
        bv[b][i] = bc[m];
        uv[b][i] = ui[m];
      },
      [&](int j, auto b, auto i) {
        const int m = 2 * j + c;
        const double w = uv[b][i] * sv[b][i];
        sig += fma(v, uv[b][i], w);
        v = fma(bv[b][i] * uv[b][i], v, -(double)(2 * m) * w);
        F[2 * m] = v;
        sf += v;
      });
  *sumF = sf;
  return sig;
}

__device__ __forceinline__ double2 operator*(double s, double2 v) { return make_double2(s * v.x, s * v.y); }
__device__ __forceinline__ double2 operator+(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 operator-(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// A chain's results per (system, parity): first flux, and q_0 (even q)
struct TauStart {
  double2 f[2], q0;
};

}  // namespace

// ---------------------------------------------------------------------------
// The solve: NP consecutive pencils per block of four wavefronts.  The
// right-hand sides are read and the state is written over the degrees (every
// access contiguous); the recurrences run one lane per (pencil, parity, real
// part), independent systems on different wavefronts, in LDS.  LDS per
// pencil: NA arrays of N complex (S and fluxes of b, then of psi; of eta; phi; g;
// 3-D: of the normal velocity) and four of N doubles (b, 1 / u of b, then of
// psi; of eta).
// ---------------------------------------------------------------------------
template <int DIM>
__global__ void __launch_bounds__(kTauThreads) tau_solve_kernel(PencilArgs a, TauFactors tf, double a0, int NP,
                                                                const double2* __restrict__ Bev,
                                                                double2* __restrict__ X) {
  constexpr int NA = DIM == 3 ? 8 : 6, S = DIM == 3 ? 9 : 7, ne = DIM == 3 ? 4 : 3;
  constexpr int eW = ne - 1;
  // state layout (p, b, u, [v], w, bz, uz, [vz], wz)
  constexpr int vP = 0, vB = 1, vU = 2, vV = 3, vW = ne, vBz = ne + 1, vUz = ne + 2, vVz = ne + 3, vWz = S - 1;
  enum { AB = 0, AZ, AE, AX, AF, AG, AT, ATZ };
  extern __shared__ double lds[];
  const int N = a.desc.N, n = N / 2, tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p0 = blockIdx.x * NP;
  // per pencil: NA complex arrays and the coefficients, padded so that the
  // pencils' lanes use different banks
  const int PS = NA * 2 * N + 4 * N + 4;
  double* inv = lds;                          // 1 / m, m <= N
  TauStart* starts = (TauStart*)(inv + N + 2);  // [NP][4]: b, the normal velocity, eta, psi
  double* sums = (double*)(starts + 4 * NP);  // [NP][parity][part]: sum of psi's particular fluxes
  double* base = sums + 4 * NP;
  for (int m = tid; m <= N; m += kTauThreads) inv[m] = m ? 1.0 / (double)m : 0.0;
  auto arr = [&](int i, int which) { return (double2*)(base + (size_t)i * PS) + which * N; };
  auto coef = [&](int i, int which) { return base + (size_t)i * PS + NA * 2 * N + which * N; };
  struct Pen {
    int slot;
    double k, cx, cy;
    bool mean;
  };
  auto pen = [&](int p) {
    Pen q;
    q.slot = p < a.P ? tf.slot[p] : -1;
    q.k = q.slot >= 0 ? tf.scal[(size_t)q.slot * kTauScal + kScK] : 0.0;
    q.cx = 1.0;
    q.cy = 0.0;
    q.mean = q.k == 0.0;
    if (DIM == 3 && q.slot >= 0 && !q.mean) {
      const int iy = p / a.Px, ix = p - iy * a.Px;
      const int ky = iy < (a.Ny + 1) / 2 ? iy : iy - a.Ny;
      q.cx = a.two_pi_over_Lx * (double)ix / q.k;
      q.cy = a.two_pi_over_Ly * (double)ky / q.k;
    }
    return q;
  };
  auto rhs = [&](int p, int e, int m) -> double2 {  // row m of evolved equation e
    return m <= N - 2 ? Bev[((size_t)p * ne + e) * N + m] : make_double2(0.0, 0.0);
  };
  const int per = kTauArrays * N;
  // b_m and 1 / u_m of a system into the coefficient arrays w, w + 1; returns
  // ratio_{m+2}
  auto coefs = [&](const double* T, int sys, double x, int i, int w, int m) {
    const double r2 = m + 2 < N ? T[(3 * sys + kRatio) * N + m + 2] : 1.0;
    coef(i, w)[m] = m + 1 < N ? 0.125 * x * inv[m + 1] * r2 : 0.0;
    coef(i, w + 1)[m] = T[(3 * sys + kUi) * N + m];
    return r2;
  };
  __syncthreads();

  // ---- right-hand sides of b, the normal velocity and phi ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    const Pen q = pen(p);
    if (q.slot < 0) continue;
    const double* T = tf.tab + (size_t)q.slot * per;
    const double k2 = q.k * q.k, i4 = 0.25 * inv[m + 1];
    const double2 fb = rhs(p, 0, m);
    double2 fu = rhs(p, 1, m);
    const double rb = coefs(T, 0, (a0 + a.kappa * k2) / a.kappa, i, 0, m);
    const double rn = coefs(T, 1, (a0 + a.nu * k2) / a.nu, i, 2, m);
    arr(i, AB)[m] = (rb * i4 / a.kappa) * fb;
    if (DIM == 3) {
      const double2 fv = rhs(p, 2, m);
      arr(i, AT)[m] = (rn * i4 / a.nu) * (q.cx * fv - q.cy * fu);
      fu = q.cx * fu + q.cy * fv;
    }
    // U = i u_L: its row is i times that of u_L; phi_m = 2 row_m + phi_{m+2}
    arr(i, AF)[m] = (m ? 2.0 : 1.0) * make_double2(-fu.y, fu.x);
    arr(i, AG)[m] = rhs(p, eW, m);
  }
  __syncthreads();

  // ---- serial: b; the normal velocity; phi ----
  const int li = lane >> 2, c = (lane >> 1) & 1, part = lane & 1;
  const Pen lq = pen(p0 + li);
  const bool lane_on = li < NP && lq.slot >= 0;
  const double* lsc = tf.scal + (size_t)(lane_on ? lq.slot : 0) * kTauScal;
  // system sys in arrays (s, f) with coefficients w: the chain, its first flux
  // and q_0 for the boundary sum G
  auto chain = [&](int s, int f, int w, int sys, int slot, double G) {
    double* Sp = (double*)arr(li, s) + part;
    const double* h = lsc + kScSys + 3 * sys;
    double sf;
    const double sig = tau_chain(Sp, (double*)arr(li, f) + part, coef(li, w), coef(li, w + 1), n, c, &sf);
    const double st = first_flux(c, G, sig, Sp[0], h);
    double* o = (double*)(starts + li * 4 + slot);
    o[2 * c + part] = st;
    if (c == 0) o[4 + part] = G - sig - h[0] * st;
    return sf;
  };
  if (lane_on && wv == 0)
    chain(AB, AZ, 0, 0, 0, lq.mean && part == 0 ? 0.5 * (a.b_top + (c ? -a.b_bottom : a.b_bottom)) : 0.0);
  if (DIM == 3 && lane_on && wv == 1) chain(AT, ATZ, 2, 1, 1, 0.0);
  if (lane_on && wv == 2) {
    double* f = (double*)arr(li, AF) + part;
    double z = 0.0, fv[2][kTauCH];
    tau_pass<true>(
        n, [&](int j, auto b, auto i) { fv[b][i] = f[2 * (2 * j + c)]; },
        [&](int j, auto b, auto i) {
          const int m = 2 * j + c;
          z = m ? z + fv[b][i] : fma(0.5, z, fv[b][i]);
          f[2 * m] = z;
        });
  }
  __syncthreads();

  // flux F_m (m >= 0) and q_m, qz_m of a system: particular plus first flux
  // times homogeneous
  auto flux = [&](const double2* F, const TauStart& s, const double* ph, int m) {
    return F[m] + ph[m] * (m & 1 ? s.f[1] : s.f[0]);
  };
  auto q_of = [&](const double2* Sa, const double2* F, const TauStart& s, const double* T, int sys, double ui, int m) {
    if (m == 0) return s.q0;
    const double2 below = m == 1 ? s.f[1] : flux(F, s, T + (3 * sys + kPh) * N, m - 2);
    return ui * (below + Sa[m]);
  };
  auto qz_of = [&](const double2* F, const TauStart& s, const double* T, int sys, int m) {
    return m == 0 ? s.f[1] : 2.0 * flux(F, s, T + (3 * sys + kPh) * N, m - 1);
  };

  // ---- b and b_z leave; g = row of w + buoyancy C b ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    const Pen q = pen(p);
    if (q.slot < 0) continue;
    const double* T = tf.tab + (size_t)q.slot * per;
    const TauStart& s = starts[i * 4];
    const double2 *Sa = arr(i, AB), *F = arr(i, AZ);
    const double* ui = coef(i, 1);
    const double2 b = q_of(Sa, F, s, T, 0, ui[m], m);
    X[((size_t)p * S + vB) * N + m] = b;
    X[((size_t)p * S + vBz) * N + m] = qz_of(F, s, T, 0, m);
    if (m <= N - 2) {
      double2 cb = cfac(m) * b;
      if (m + 2 < N) cb = cb - 0.5 * q_of(Sa, F, s, T, 0, ui[m + 2], m + 2);
      arr(i, AG)[m] = arr(i, AG)[m] + a.buoyancy * cb;
    }
  }
  __syncthreads();

  // f_m / (4 nu (m + 1)) of eta with f_m = k g_m + 2 (m + 1) phi_{m+1}, m <= N - 2
  auto fh_eta = [&](int i, double k, int m) {
    return (1.0 / a.nu) * (0.25 * k * inv[m + 1] * arr(i, AG)[m] + 0.5 * arr(i, AF)[m + 1]);
  };
  // ---- right-hand side of eta ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    const Pen q = pen(p);
    if (q.slot < 0) continue;
    const double* T = tf.tab + (size_t)q.slot * per;
    const double r2 = m + 2 < N ? T[(3 + kRatio) * N + m + 2] : 1.0;
    arr(i, AE)[m] = m <= N - 2 ? r2 * fh_eta(i, q.k, m) : make_double2(0.0, 0.0);
  }
  __syncthreads();

  // ---- serial: eta with zero wall values ----
  if (lane_on && wv == 0) chain(AE, AX, 2, 1, 2, 0.0);
  __syncthreads();

  // ---- right-hand side of psi ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    const Pen q = pen(p);
    if (q.slot < 0) continue;
    const double* T = tf.tab + (size_t)q.slot * per;
    const TauStart& s = starts[i * 4 + 2];
    const double2 *Sa = arr(i, AE), *F = arr(i, AX);
    const double k2 = q.k * q.k, al = a0 + a.nu * k2, d = (double)(m + 1);
    const double r2 = coefs(T, 2, k2, i, 0, m);
    double2 ce = make_double2(0.0, 0.0);
    if (m <= N - 2) {
      // C eta, from al C eta = f + nu D zeta where the differences of eta cancel
      if (al > 4.0 * a.nu * d * d) {
        ce = (4.0 * a.nu * d / al) * (fh_eta(i, q.k, m) + flux(F, s, T + (3 + kPh) * N, m));
      } else {
        const double* ui = coef(i, 3);
        ce = cfac(m) * q_of(Sa, F, s, T, 1, ui[m], m);
        if (m + 2 < N) ce = ce - 0.5 * q_of(Sa, F, s, T, 1, ui[m + 2], m + 2);
      }
    }
    arr(i, AB)[m] = (0.25 * r2 * inv[m + 1]) * ce;
  }
  __syncthreads();

  // ---- serial: psi ----
  if (lane_on && wv == 0) sums[li * 4 + c * 2 + part] = chain(AB, AZ, 0, 2, 3, 0.0);
  __syncthreads();

  // wall vorticity t of either class from sum U = 0; U0: the mean pencil's free
  // constant of U
  auto walls = [&](const Pen& q, int i, const double* T, double2* t, double2* U0) {
    const double* sc = tf.scal + (size_t)q.slot * kTauScal;
    const TauStart &s = starts[i * 4 + 3], &se = starts[i * 4 + 2];
    *U0 = make_double2(0.0, 0.0);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const double2 sf = make_double2(sums[i * 4 + e * 2], sums[i * 4 + e * 2 + 1]);
      double2 su = -2.0 * (sf + sc[kScPh + e] * s.f[e]);
      if (e == 1) su = su - s.f[1];
      if (q.mean && e == 1) {  // s_0 = a0 U_0 with sum U = 0
        const double den = T[kHs * N] - a0 * (T[kHu * N] - sc[kScU + 1]);
        const double2 r = arr(i, AF)[0] + a.nu * se.f[1] + a0 * (s.f[1] + su);
        t[1] = (-1.0 / den) * r;
        *U0 = -1.0 * su - sc[kScU + 1] * t[1];
      } else {
        t[e] = (-1.0 / sc[kScU + e]) * su;
      }
    }
  };
  // ---- eta and psi in place of their S ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    const Pen q = pen(p);
    if (q.slot < 0) continue;
    const double* T = tf.tab + (size_t)q.slot * per;
    double2 t[2], U0;
    walls(q, i, T, t, &U0);
    const double2 te = m & 1 ? t[1] : t[0];
    arr(i, AE)[m] = q_of(arr(i, AE), arr(i, AX), starts[i * 4 + 2], T, 1, coef(i, 3)[m], m) + T[kHe * N + m] * te;
    arr(i, AB)[m] = q_of(arr(i, AB), arr(i, AZ), starts[i * 4 + 3], T, 2, coef(i, 1)[m], m) + T[kHp * N + m] * te;
  }
  __syncthreads();

  // ---- velocity and pressure ----
  for (int idx = tid; idx < NP * N; idx += kTauThreads) {
    const int i = idx / N, m = idx - i * N, p = p0 + i;
    if (p >= a.P) continue;
    const Pen q = pen(p);
    double2* Xp = X + (size_t)p * S * N + m;
    if (q.slot < 0) {
#pragma unroll
      for (int v = 0; v < S; ++v) Xp[v * N] = make_double2(0.0, 0.0);
      continue;
    }
    const double* T = tf.tab + (size_t)q.slot * per;
    const double2 *psi = arr(i, AB), *eta = arr(i, AE), *g = arr(i, AG);
    const double k = q.k;
    double2 t[2], U0;
    walls(q, i, T, t, &U0);
    const double2 to = m & 1 ? t[0] : t[1];  // of the class of U, p and s at this degree
    double2 U = T[kHu * N + m] * to - qz_of(arr(i, AZ), starts[i * 4 + 3], T, 2, m);
    if (m == 0) U = U + U0;
    const double2 w = k * psi[m], uz = eta[m] - k * w;
    // pressure: D p from the w rows where the degree exceeds k / 2, else from s
    double2 pr = make_double2(0.0, 0.0);
    if (m >= 1 && k < 2.0 * m) {
      const int l = m - 1;
      double2 ce = cfac(l) * eta[l], cp = cfac(l) * psi[l];
      if (l + 2 < N) {
        ce = ce - 0.5 * eta[l + 2];
        cp = cp - 0.5 * psi[l + 2];
      }
      pr = 0.5 * inv[m] * (g[l] - (a0 * k) * cp - (a.nu * k) * ce);
    } else if (!q.mean) {
      const double2 s = arr(i, AF)[m] + a.nu * qz_of(arr(i, AX), starts[i * 4 + 2], T, 1, m) + T[kHs * N + m] * to;
      pr = (1.0 / k) * (a0 * U - s);
    } else {  // m = 0: gauge p(1) = 0 of the mean pencil
#pragma unroll 8
      for (int l = 1; l < N; ++l) pr = pr - 0.5 * inv[l] * g[l - 1];
    }
    Xp[vP * N] = pr;
    Xp[vW * N] = w;
    Xp[vWz * N] = (-k) * U;
    // u_L = -i U
    const double2 ul = make_double2(U.y, -U.x), uzl = make_double2(uz.y, -uz.x);
    if (DIM == 3) {
      const TauStart& s = starts[i * 4 + 1];
      const double2 T0 = q_of(arr(i, AT), arr(i, ATZ), s, T, 1, coef(i, 3)[m], m);
      const double2 Tz = qz_of(arr(i, ATZ), s, T, 1, m);
      Xp[vU * N] = q.cx * ul - q.cy * T0;
      Xp[vV * N] = q.cy * ul + q.cx * T0;
      Xp[vUz * N] = q.cx * uzl - q.cy * Tz;
      Xp[vVz * N] = q.cy * uzl + q.cx * Tz;
    } else {
      Xp[vU * N] = ul;
      Xp[vUz * N] = uzl;
    }
  }
}

// ---------------------------------------------------------------------------
// Launches
// ---------------------------------------------------------------------------
static void allow_lds(const void* fn, size_t bytes) {
  if (bytes > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

static size_t tau_lds_bytes(int dim, int N, int NP) {
  const size_t pencil = ((dim == 3 ? 8 : 6) * 2 * N + 4 * N + 4) * sizeof(double) + 4 * sizeof(TauStart) +
                        4 * sizeof(double);
  return NP * pencil + (size_t)(N + 2) * sizeof(double);
}

hipError_t launch_tau_factor(const PencilArgs& a, double a0, const TauFactors& tf, hipStream_t st) {
  const int N = a.desc.N;
  // six lanes per wavenumber, at most half a compute unit's LDS per block
  const size_t per = (size_t)(kTauArrays * N + kTauScal + 2) * sizeof(double);
  const int KB = (int)std::max<size_t>(1, std::min<size_t>(8, (size_t)(80 * 1024) / per));
  const size_t lds = KB * per;
  allow_lds((const void*)tau_factor_kernel, lds);
  hipLaunchKernelGGL(tau_factor_kernel, dim3((tf.nk + KB - 1) / KB), dim3(kWave), lds, st, N, tf.nk, KB, a0, a.kappa,
                     a.nu, tf.k, tf.tab, tf.scal);
  return hipGetLastError();
}

template <int DIM>
static hipError_t launch_tau_solve_t(const PencilArgs& a, const TauFactors& tf, double a0, const void* Bev, void* X,
                                     hipStream_t st) {
  const int N = a.desc.N;
  // pencils per block: as many as leave two blocks per compute unit, both in
  // LDS (80 KB each) and in number
  int NP = 8;
  while (NP > 1 && (tau_lds_bytes(DIM, N, NP) > 80 * 1024 || (a.P + NP - 1) / NP < 2 * tf.cus)) NP >>= 1;
  const size_t lds = tau_lds_bytes(DIM, N, NP);
  allow_lds((const void*)tau_solve_kernel<DIM>, lds);
  hipLaunchKernelGGL(tau_solve_kernel<DIM>, dim3((a.P + NP - 1) / NP), dim3(kTauThreads), lds, st, a, tf, a0, NP,
                     (const double2*)Bev, (double2*)X);
  return hipGetLastError();
}

hipError_t launch_tau_solve(const PencilArgs& a, const TauFactors& tf, double a0, const void* Bev, void* X,
                            hipStream_t st) {
  return a.desc.dim == 3 ? launch_tau_solve_t<3>(a, tf, a0, Bev, X, st)
                         : launch_tau_solve_t<2>(a, tf, a0, Bev, X, st);
}

}  // namespace stau
