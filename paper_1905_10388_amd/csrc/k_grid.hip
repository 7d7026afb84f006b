// Grid <-> coefficient transforms of selected state variables (Sec. VI "Data
// manipulation": a field's grid data and its coefficient data; Sec. IV
// "Scaled transforms & dealiasing": grids at scale 1 or 3/2), and their
// adjoints.  The z and y stages reuse the step's transform kernels; this file
// holds the x stage on the caller's grid layout.
//
// Grid layout (real float64): g[f][ix][l][jz] (2-D: g[f][ix][jz]), with
// ix < Lg = scale Nx, l < scale Ny, jz < Mg = scale Nz on the ascending
// Chebyshev Gauss grid; spectral rows (complex) s[f][jz][l][kx], kx < Px.
//
//   DIR +1 (x synthesis): g = s0 Re c_0 + 2 s1 Re sum_{1 <= k < Pa} c_k e^{2 pi i k ix / Lg}
//   DIR -1 (x analysis):  c_0 = s0 sum_ix g,  c_k = s1 sum_ix g e^{-2 pi i k ix / Lg}  (k < Pa),
//                         c_k = 0 for Pa <= k < Px
//
// The synthesis at s0 = s1 = 1 is the complex-to-real transform of the half
// spectrum (Nyquist and padding zero); the analysis at s0 = s1 = 1 / Lg is the
// truncating forward transform.  Their adjoints under the real inner product
// (complex coefficients as pairs of reals) are the analysis with s0 = 1,
// s1 = 2 and the synthesis with s0 = 1 / Lg, s1 = 1 / (2 Lg).
//
// One block transforms TZ consecutive z levels of one (field, y level): the
// grid values of a fixed ix are TZ contiguous doubles, and two real rows are
// packed into each complex FFT (TZ / 2 sequences of Lg points in LDS).
#include "fft.h"
#include "xform.h"

namespace stau {

namespace {

constexpr int kGThreads = 256;
constexpr int kGMaxBF = 6;          // butterflies per thread per radix-4 pass
constexpr int kGMaxPoints = 6144;   // (TZ / 2) * Lg complex points per block

template <int DIR>
__global__ void __launch_bounds__(kGThreads) xgrid_kernel(XformArgs a, int Lg, int Ngy, int Mg,
                                                          const double2* __restrict__ tw,
                                                          const void* __restrict__ in,
                                                          void* __restrict__ out, double s0,
                                                          double s1, int TZ) {
  extern __shared__ double2 smem[];
  cd* buf = (cd*)smem;
  const int jz0 = blockIdx.x * TZ, l = blockIdx.y, f = blockIdx.z;
  const int Pa = a.Pa, Px = a.Px, tid = threadIdx.x;
  const int half = TZ / 2;
  auto grow = [&](int ix) { return (((size_t)f * Lg + ix) * Ngy + l) * Mg + jz0; };
  auto srow = [&](int t) { return (((size_t)f * Mg + jz0 + t) * Ngy + l) * Px; };
  if constexpr (DIR > 0) {
    const double2* S = (const double2*)in;
    double* g = (double*)out;
    for (int idx = tid; idx < half * Lg; idx += kGThreads) {
      const int s = idx / Lg, k = idx - s * Lg;
      const int kk = k < Pa ? k : (k > Lg - Pa ? Lg - k : -1);
      cd z = mk(0.0, 0.0);
      if (kk >= 0) {
        const double2 A = S[srow(2 * s) + kk], B = S[srow(2 * s + 1) + kk];
        const double w = kk == 0 ? s0 : s1;
        cd Ak = mk(w * A.x, kk == 0 ? 0.0 : w * A.y), Bk = mk(w * B.x, kk == 0 ? 0.0 : w * B.y);
        // rows A, B packed as A + i B: positive frequencies A_k + i B_k,
        // negative ones conj(A_k) + i conj(B_k)
        z = k < Pa ? mk(Ak.x - Bk.y, Ak.y + Bk.x) : mk(Ak.x + Bk.y, Bk.x - Ak.y);
      }
      buf[idx] = z;
    }
    __syncthreads();
    fft_lds<+1, kGMaxBF>(buf, Lg, half, (const cd*)tw, tid, kGThreads);
    for (int idx = tid; idx < TZ * Lg; idx += kGThreads) {
      const int ix = idx / TZ, t = idx - ix * TZ;
      const cd v = buf[(t >> 1) * Lg + ix];
      g[grow(ix) + t] = (t & 1) ? v.y : v.x;
    }
  } else {
    const double* g = (const double*)in;
    double2* S = (double2*)out;
    double* bd = (double*)smem;
    for (int idx = tid; idx < TZ * Lg; idx += kGThreads) {
      const int ix = idx / TZ, t = idx - ix * TZ;
      bd[2 * ((t >> 1) * Lg + ix) + (t & 1)] = g[grow(ix) + t];
    }
    __syncthreads();
    fft_lds<-1, kGMaxBF>(buf, Lg, half, (const cd*)tw, tid, kGThreads);
    for (int idx = tid; idx < TZ * Px; idx += kGThreads) {
      const int t = idx / Px, k = idx - t * Px;
      double2 v = make_double2(0.0, 0.0);
      if (k < Pa) {
        const cd Z = buf[(t >> 1) * Lg + k], Zm = buf[(t >> 1) * Lg + (k == 0 ? 0 : Lg - k)];
        // unpack: A_k = (Z_k + conj Z_{-k}) / 2, B_k = (Z_k - conj Z_{-k}) / (2 i)
        const cd A = mk(0.5 * (Z.x + Zm.x), 0.5 * (Z.y - Zm.y));
        const cd B = mk(0.5 * (Z.y + Zm.y), -0.5 * (Z.x - Zm.x));
        const cd c = (t & 1) ? B : A;
        const double w = k == 0 ? s0 : s1;
        v = make_double2(w * c.x, w * c.y);
      }
      S[srow(t) + k] = v;
    }
  }
}

// A pair of grid values of the caller's array, which is aligned to its doubles only
struct __attribute__((aligned(8))) GridPair {
  double x, y;
};

// The same at the compile-time padded lengths L = 3 Nx / 2, registers to registers
// (fft_block): NSQ pairs of z levels per block, entries of the half spectra
// read and written along k, grid values along z.  The synthesis forms the packed
// spectrum in its first stage's inputs (the middle third is zero); in the last
// stage of the analysis a thread does the butterflies j and W - j, which hold
// an entry and its conjugate partner.  Bound by the memory (128x128x64, four
// fields, 190 MB: synthesis 67 -> 39 us, analysis 75 -> 33 us against
// xgrid_kernel, whose index divisions and LDS passes took as long again).
template <typename PL, int NSQ, int NT>
__global__ void __launch_bounds__(NT) xsynth_kernel(XformArgs a, int Ngy, int Mg, const double2* __restrict__ S,
                                                    double* __restrict__ g, double s0, double s1) {
  extern __shared__ double2 smem[];
  constexpr int L = PL::L, Pa = L / 3, Px = Pa + 1, R0 = PL::r[0], W = L / R0, RL = PL::PT;
  static_assert(R0 % 3 == 0, "thirds of the first stage");
  const int jz0 = blockIdx.x * 2 * NSQ, l = blockIdx.y, f = blockIdx.z, tid = threadIdx.x;
  auto load = [&](int, int s, int j, cd* v) {
    const int jz = jz0 + 2 * s;
    const double2* A = S + (((size_t)f * Mg + jz) * Ngy + l) * Px;
    const double2* B = A + (size_t)Ngy * Px;
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      v[r] = mk(0.0, 0.0);
      if (3 * r >= R0 && 3 * r < 2 * R0) continue;  // padding
      const bool up = 3 * r >= R0;
      const int k = j + r * W, kk = up ? L - k : k;
      if (jz >= Mg || kk >= Pa) continue;
      cd Ak = ld2(A + kk), Bk = ld2(B + kk);
      const double w = kk == 0 ? s0 : s1;
      Ak = mk(w * Ak.x, kk == 0 ? 0.0 : w * Ak.y);
      Bk = mk(w * Bk.x, kk == 0 ? 0.0 : w * Bk.y);
      v[r] = up ? mk(Ak.x + Bk.y, Bk.x - Ak.y) : mk(Ak.x - Bk.y, Ak.y + Bk.x);
    }
  };
  auto store = [&](int s, int j, cd* v) {
    const int jz = jz0 + 2 * s;
    if (jz >= Mg) return;
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int ix = j + r * (L / RL);
      *(GridPair*)(g + (((size_t)f * L + ix) * Ngy + l) * Mg + jz) = GridPair{v[r].x, v[r].y};
    }
  };
  fft_block<PL, +1, NSQ, NT, false, true, true, double>((cd*)smem, (const cd*)a.twx, tid, load, store,
                                                         [](int s, int i) { return s * (L + 1) + i; });
}

template <typename PL, int NSQ, int NT>
__global__ void __launch_bounds__(NT) xanal_kernel(XformArgs a, int Ngy, int Mg, const double* __restrict__ g,
                                                   double2* __restrict__ S, double s0, double s1) {
  extern __shared__ double2 smem[];
  constexpr int L = PL::L, Pa = L / 3, Px = Pa + 1, R0 = PL::r[0], RL = PL::PT, W = L / RL, U = W / 2;
  static_assert(RL % 3 == 0 && NSQ * U <= NT, "thirds of the last stage, one pair of butterflies per thread");
  cd* buf = (cd*)smem;
  const int jz0 = blockIdx.x * 2 * NSQ, l = blockIdx.y, f = blockIdx.z, tid = threadIdx.x;
  auto load = [&](int, int s, int j, cd* v) {
    const int jz = jz0 + 2 * s;
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      v[r] = mk(0.0, 0.0);
      if (jz >= Mg) continue;
      const GridPair q = *(const GridPair*)(g + (((size_t)f * L + j + r * (L / R0)) * Ngy + l) * Mg + jz);
      v[r] = mk(q.x, q.y);
    }
  };
  auto at = [](int s, int i) { return s * (L + 1) + i; };
  fft_block<PL, -1, NSQ, NT, true, true, false, double>(buf, (const cd*)a.twx, tid, load, [](int, int, cd*) {}, at);
  const int s = tid / U, t = tid - s * U, jz = jz0 + 2 * s;
  if (s >= NSQ || jz >= Mg) return;
  const int j1 = t, j2 = t ? W - t : U;
  cd v1[RL], v2[RL];
#pragma unroll
  for (int q = 0; q < RL; ++q) {
    v1[q] = buf[at(s, j1 + q * W)];
    v2[q] = buf[at(s, j2 + q * W)];
  }
  fft_butterfly<L, RL, W, -1, double>(v1, j1, (const cd*)a.twx);
  fft_butterfly<L, RL, W, -1, double>(v2, j2, (const cd*)a.twx);
  double2* SA = S + (((size_t)f * Mg + jz) * Ngy + l) * Px;
  double2* SB = SA + (size_t)Ngy * Px;
  auto put = [&](int k, cd Z, cd Zm) {  // A_k = (Z_k + conj Z_{-k}) / 2, B_k = (Z_k - conj Z_{-k}) / (2 i)
    const double w = 0.5 * (k == 0 ? s0 : s1);
    st2(SA + k, mk(w * (Z.x + Zm.x), w * (Z.y - Zm.y)));
    st2(SB + k, mk(w * (Z.y + Zm.y), -w * (Z.x - Zm.x)));
  };
  auto sel = [](bool c, cd x, cd y) { return mk(c ? x.x : y.x, c ? x.y : y.y); };
#pragma unroll
  for (int q = 0; 3 * q < RL; ++q) {
    put(j1 + q * W, v1[q], sel(t, v2[RL - 1 - q], v1[q ? RL - q : 0]));
    put(j2 + q * W, v2[q], sel(t, v1[RL - 1 - q], v2[RL - 1 - q]));
  }
  if (t == 0) {
    st2(SA + Pa, mk(0.0, 0.0));
    st2(SB + Pa, mk(0.0, 0.0));
  }
}

// zero the variables of fl in X[p][var][n]
__global__ void zero_vars_kernel(int P, int S, int N, FieldList fl, double2* __restrict__ X) {
  const size_t total = (size_t)P * fl.nf * N;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const int n = (int)(i % N);
    const size_t q = i / N;
    const int f = (int)(q % fl.nf);
    const size_t p = q / fl.nf;
    X[(p * S + fl.var[f]) * N + n] = make_double2(0.0, 0.0);
  }
}

int grid_blocks(size_t total) {
  const size_t b = (total + 255) / 256;
  return (int)(b < 8192 ? (b ? b : 1) : 8192);
}

}  // namespace

bool xgrid_supported(int Lg, int Mg) {
  int TZ = 2;
  while (TZ < 16 && Mg % (2 * TZ) == 0 && TZ * Lg <= kGMaxPoints) TZ *= 2;
  return Mg % 2 == 0 && (TZ / 2) * Lg <= kGMaxPoints;
}

template <int NSQ, int NT, int... R>
static hipError_t launch_xgrid_ct(const XformArgs& a, int dir, int nf, int Ngy, int Mg, const void* in, void* out,
                                  double s0, double s1, hipStream_t st) {
  using SY = FftPlan<R...>;
  using AN = typename FftPlan<R...>::reverse;
  constexpr size_t lds = (size_t)NSQ * (SY::L + 1) * sizeof(double2);
  const dim3 grid((Mg + 2 * NSQ - 1) / (2 * NSQ), Ngy, nf);
  if (dir > 0) {
    auto fn = xsynth_kernel<SY, NSQ, NT>;
    allow_lds((const void*)fn, lds);
    hipLaunchKernelGGL(fn, grid, dim3(NT), lds, st, a, Ngy, Mg, (const double2*)in, (double*)out, s0, s1);
  } else {
    auto fn = xanal_kernel<AN, NSQ, NT>;
    allow_lds((const void*)fn, lds);
    hipLaunchKernelGGL(fn, grid, dim3(NT), lds, st, a, Ngy, Mg, (const double*)in, (double2*)out, s0, s1);
  }
  return hipGetLastError();
}

hipError_t launch_xgrid(const XformArgs& a, int dir, int nf, int Lg, int Ngy, int Mg,
                        const double2* tw, const void* in, void* out, double s0, double s1,
                        hipStream_t st) {
  if (!xgrid_supported(Lg, Mg)) return hipErrorInvalidValue;
  // the dealiased lengths of Nx = 16 .. 4096: up to eight pairs of z levels (128
  // bytes of a grid row) in 98 KB of LDS; the scale-1 lengths at run time
  if (Lg == 3 * a.Pa) switch (Lg) {
    case 24: return launch_xgrid_ct<8, 64, 6, 4>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 48: return launch_xgrid_ct<8, 64, 6, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 96: return launch_xgrid_ct<8, 128, 6, 4, 4>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 192: return launch_xgrid_ct<8, 128, 6, 8, 4>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 384: return launch_xgrid_ct<8, 256, 6, 8, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 768: return launch_xgrid_ct<4, 256, 6, 4, 4, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 1536: return launch_xgrid_ct<2, 256, 6, 4, 8, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 3072: return launch_xgrid_ct<2, 512, 6, 8, 8, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
    case 6144: return launch_xgrid_ct<1, 512, 6, 16, 8, 8>(a, dir, nf, Ngy, Mg, in, out, s0, s1, st);
  }
  // the largest power of two TZ <= 16 dividing Mg with (TZ / 2) Lg points in LDS
  int TZ = 2;
  while (TZ < 16 && Mg % (2 * TZ) == 0 && TZ * Lg <= kGMaxPoints) TZ *= 2;
  const size_t lds = (size_t)(TZ / 2) * Lg * sizeof(double2);
  const dim3 grid(Mg / TZ, Ngy, nf);
  const void* fn = dir > 0 ? (const void*)xgrid_kernel<+1> : (const void*)xgrid_kernel<-1>;
  if (lds > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (dir > 0)
    hipLaunchKernelGGL(xgrid_kernel<+1>, grid, dim3(kGThreads), lds, st, a, Lg, Ngy, Mg, tw, in, out,
                       s0, s1, TZ);
  else
    hipLaunchKernelGGL(xgrid_kernel<-1>, grid, dim3(kGThreads), lds, st, a, Lg, Ngy, Mg, tw, in, out,
                       s0, s1, TZ);
  return hipGetLastError();
}

hipError_t launch_zero_vars(int P, int S, int N, const FieldList& fl, void* X, hipStream_t st) {
  hipLaunchKernelGGL(zero_vars_kernel, dim3(grid_blocks((size_t)P * fl.nf * N)), dim3(256), 0, st, P,
                     S, N, fl, (double2*)X);
  return hipGetLastError();
}

}  // namespace stau
