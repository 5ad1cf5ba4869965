// Far field radiated by the equivalent currents of every box (Sec. II-A: the
// equivalent J and M on a fictitious surface radiate the exterior field;
// Sec. III: they are the solved unknowns).  With the point-sampled currents of
// the coupling fill (patch q of element m carries J = sum_a xJ t_qa at
// rho_q + pitch (ix, iy, 0), M likewise) and eta = 1,
//     E_theta = N . theta^ + L . phi^,   E_phi = N . phi^ - L . theta^,
//     N = sum A_q J e^{jk rhat . r'},    L = sum A_q M e^{jk rhat . r'}
// (common factor -jk e^{-jkr}/(4 pi r) dropped).  At the direction cosines of
// the bins of an Lu x Lv lattice DFT, k pitch u = 2 pi p' / Lu (p' the signed
// bin), the sum over elements is the zero-padded 2-D DFT with kernel
// e^{+j 2 pi (p ix / Lu + q iy / Lv)} of the lattice data: a Stockham pass of
// sign +1 along x (the pass of the coupling apply), then one kernel that runs
// the pass along y in LDS and projects its points onto the directions; where
// that leaves the chip idle, a pass along y and a projection by single bins.
#include <algorithm>
#include <cmath>
#include <vector>

#include "fft_device.h"

namespace emsurf {
namespace {

struct PatternArgs {
  const double2* W;      // [iy][p][r][u], transformed along x
  const double* rho;
  const double* area;
  const double* tan;
  const double2* tw;     // twiddles of the y transform
  int P, Lu, ny, nrhs;
  double pitch, k;
  double2* E;            // [r][q][p][2] (E_theta, E_phi), upper half space; or NULL
  double* U;             // [r][half space][q][p] radiation intensity; or NULL
  double* part;          // [r][parts] partial powers, with U
};

// One workgroup per (x bin p, right-hand side r), which owns the bins (q, p)
// of all q.  It takes BT / 4 patches at a time: their 2 J and 2 M columns are
// transformed along y in LDS (Lv points), then every thread adds the patches to
// its bins, the upper half space (HS = 1, for E) or both at once (HS = 2, for
// U).  A spectrum written by a y pass and read by a projection of each half
// space is 403 MB at 64 x 57 elements, n_eq 192, 2 RHS and 256 x 256 bins: 330
// of 375 us per call, now 97 of 137 us (bound by the FP64 sums of two
// workgroups per CU, whose spectra fill the LDS).  With a patch's phase split
// into e^{jkux} (per workgroup), e^{jkvy} and e^{jkwz} (kept while the next
// patch has the same y or z) the sums need few sincos:
//   S = (t . (cp, sp, 0) J, t_z st J, t . phi^ J) summed over the tangents,
//   R the same of M,
//   E_theta += e^{jk..} (+-w S0 - S1 + R2),  E_phi += e^{jk..} (S2 -+ w R0 + R1)
// with theta^ = (+-w cp, +-w sp, -st) above and below.  Bins outside the
// visible region u^2 + v^2 < 1 are zero.
template <int L, int HS>
__global__ void __launch_bounds__((Shape<L, 1>::NT)) pattern_kernel(PatternArgs a) {
  using SH = Shape<L, 1>;
  constexpr int BT = SH::BT, NT = SH::NT, NBIN = (L + NT - 1) / NT, PC = BT / 4;
  static_assert(BT % 4 == 0, "whole patches");
  __shared__ double2 lds[L * BT];
  __shared__ double2 phx[PC];
  __shared__ double red[NT];
  const int t = threadIdx.x, p = blockIdx.x, r = blockIdx.y, n = 4 * a.P;
  const double pi = 3.14159265358979323846;
  const int ps = p < (a.Lu + 1) / 2 ? p : p - a.Lu;
  const double u = 2.0 * pi * ps / (a.Lu * a.k * a.pitch);
  struct Bin {
    double v, w, cp, sp, st;
    double2 py, pz;               // e^{jkvy}, e^{jkwz}
    double2 et[HS], ep[HS];       // above, below
    bool vis;
  } bin[NBIN];
#pragma unroll
  for (int j = 0; j < NBIN; ++j) {
    const int q = t + NT * j, qs = q < (L + 1) / 2 ? q : q - L;
    Bin& B = bin[j];
    B.v = 2.0 * pi * qs / (L * a.k * a.pitch);
    const double s2 = u * u + B.v * B.v;
    B.vis = q < L && s2 < 1.0;
    B.w = B.vis ? sqrt(1.0 - s2) : 1.0;
    B.st = sqrt(s2);
    B.cp = B.st > 0.0 ? u / B.st : 1.0;
    B.sp = B.st > 0.0 ? B.v / B.st : 0.0;
    B.py = B.pz = double2{1.0, 0.0};
#pragma unroll
    for (int h = 0; h < HS; ++h) B.et[h] = B.ep[h] = double2{0.0, 0.0};
  }
  if (u * u < 1.0) {   // (the whole workgroup)
    PassArgs f{};
    f.n_in = a.ny;
    f.n_out = L;
    f.in_pt = a.Lu * a.nrhs * n;
    f.sign = +1;
    f.scale = 1.0;
    const double2* Wl = a.W + ((long long)p * a.nrhs + r) * n;
    double y0 = 0.0, z0 = 0.0;   // of the phases kept in bin (e^0 = 1)
    const int b = t % BT, g = t / BT;
    for (int pb = 0; pb < a.P; pb += PC) {
      // column b: J of patch pb + b / 2 (b < BT / 2), then M
      const int h = b < BT / 2 ? 0 : 1, cl = 2 * pb + b - h * (BT / 2);
      run_stage<L, 1, 0, 0, 1, double2, double2, double2, true>(f, lds, Wl + h * 2 * a.P + cl, nullptr, a.tw,
                                                                cl < 2 * a.P, b, g, GreenGen{}, 0, 0);
      if (t < PC && pb + t < a.P) {
        double sn, cs;
        sincos(a.k * u * a.rho[3 * (pb + t)], &sn, &cs);
        phx[t] = double2{a.area[pb + t] * cs, a.area[pb + t] * sn};
      }
      __syncthreads();
      const int np = a.P - pb < PC ? a.P - pb : PC;
      for (int i = 0; i < np; ++i) {
        const double* rho = a.rho + 3 * (pb + i);
        const double* t0 = a.tan + 6 * (pb + i);
        const double y = rho[1], z = rho[2];
        const bool ny = y != y0, nz = z != z0;
        y0 = y;
        z0 = z;
#pragma unroll
        for (int j = 0; j < NBIN; ++j) {
          Bin& B = bin[j];
          const int q = t + NT * j < L ? t + NT * j : 0;
          if (ny) sincos(a.k * B.v * y, &B.py.y, &B.py.x);
          if (nz) sincos(a.k * B.w * z, &B.pz.y, &B.pz.x);
          const double2 pxy = cmul(phx[i], B.py);
          const double2 up = cmul(pxy, B.pz), dn = cmul(pxy, double2{B.pz.x, -B.pz.y});
          double2 S[2][3];
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const double2 x0 = lds[lds_column<L, 1>(q, m * (BT / 2) + 2 * i)];
            const double2 x1 = lds[lds_column<L, 1>(q, m * (BT / 2) + 2 * i + 1)];
            const double e0 = t0[0] * B.cp + t0[1] * B.sp, e1 = t0[3] * B.cp + t0[4] * B.sp;
            const double g0 = t0[2] * B.st, g1 = t0[5] * B.st;
            const double f0 = t0[1] * B.cp - t0[0] * B.sp, f1 = t0[4] * B.cp - t0[3] * B.sp;
            S[m][0] = double2{B.w * (e0 * x0.x + e1 * x1.x), B.w * (e0 * x0.y + e1 * x1.y)};
            S[m][1] = double2{g0 * x0.x + g1 * x1.x, g0 * x0.y + g1 * x1.y};
            S[m][2] = double2{f0 * x0.x + f1 * x1.x, f0 * x0.y + f1 * x1.y};
          }
          // theta: w S0 - S1 + R2 above, -w S0 - S1 + R2 below; phi: S2 - w R0 + R1 above, S2 + w R0 + R1 below
          const double2 ct{S[1][2].x - S[0][1].x, S[1][2].y - S[0][1].y};
          const double2 cf{S[0][2].x + S[1][1].x, S[0][2].y + S[1][1].y};
          B.et[0] = cadd(B.et[0], cmul(up, cadd(ct, S[0][0])));
          B.ep[0] = cadd(B.ep[0], cmul(up, csub(cf, S[1][0])));
          if constexpr (HS == 2) {
            B.et[1] = cadd(B.et[1], cmul(dn, csub(ct, S[0][0])));
            B.ep[1] = cadd(B.ep[1], cmul(dn, cadd(cf, S[1][0])));
          }
        }
      }
      __syncthreads();   // every column is read before the next ones arrive
    }
  }
  const double du = 2.0 * pi / (a.Lu * a.k * a.pitch), dv = 2.0 * pi / (L * a.k * a.pitch);
  double power = 0.0;
#pragma unroll
  for (int j = 0; j < NBIN; ++j) {
    const Bin& B = bin[j];
    const int q = t + NT * j;
    if (q >= L) continue;
    if constexpr (HS == 1) {
      double2* out = a.E + (((long long)r * L + q) * a.Lu + p) * 2;
      out[0] = B.vis ? B.et[0] : double2{0.0, 0.0};
      out[1] = B.vis ? B.ep[0] : double2{0.0, 0.0};
    }
    if constexpr (HS == 2) {
#pragma unroll
      for (int h = 0; h < HS; ++h) {
        const double U = B.vis ? B.et[h].x * B.et[h].x + B.et[h].y * B.et[h].y + B.ep[h].x * B.ep[h].x +
                                     B.ep[h].y * B.ep[h].y
                               : 0.0;
        a.U[(((long long)r * 2 + h) * L + q) * a.Lu + p] = U;
        power += U * du * dv / B.w;
      }
    }
  }
  if constexpr (HS == 1) return;
  red[t] = power;
  __syncthreads();
  if (t < 64) {   // (fixed order: lane t adds its share, then a tree)
    double s = 0.0;
    for (int i = t; i < NT; i += 64) s += red[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (t == 0) a.part[(long long)r * a.Lu + p] = s;
  }
}

// The projection by single bins: one thread per bin (q, p) of the spectrum
// a.W = X[q][p][r][u]; grid (blocks of BIN_THREADS bins, r).
constexpr int BIN_THREADS = 256;
template <int HS> __global__ void __launch_bounds__(BIN_THREADS) bins_kernel(PatternArgs a, int Lv) {
  __shared__ double red[BIN_THREADS];
  const int r = blockIdx.y, n = 4 * a.P;
  const long long bins = (long long)Lv * a.Lu, bin = blockIdx.x * (long long)BIN_THREADS + threadIdx.x;
  const int p = (int)(bin % a.Lu), q = (int)(bin / a.Lu);
  const double pi = 3.14159265358979323846;
  const int ps = p < (a.Lu + 1) / 2 ? p : p - a.Lu, qs = q < (Lv + 1) / 2 ? q : q - Lv;
  const double u = 2.0 * pi * ps / (a.Lu * a.k * a.pitch), v = 2.0 * pi * qs / (Lv * a.k * a.pitch);
  const double s2 = u * u + v * v;
  const bool vis = bin < bins && s2 < 1.0;
  double power = 0.0;
#pragma unroll
  for (int h = 0; h < HS; ++h) {
    double2 et{0.0, 0.0}, ep{0.0, 0.0};
    if (vis) {
      const double w = h == 0 ? sqrt(1.0 - s2) : -sqrt(1.0 - s2), st = sqrt(s2);
      const double cp = st > 0.0 ? u / st : 1.0, sp = st > 0.0 ? v / st : 0.0;
      const double2* xb = a.W + (bin * a.nrhs + r) * n;
      double2 N[3] = {}, M[3] = {};
      for (int i = 0; i < a.P; ++i) {
        double sn, cs;
        sincos(a.k * (u * a.rho[3 * i] + v * a.rho[3 * i + 1] + w * a.rho[3 * i + 2]), &sn, &cs);
        const double2 ph{a.area[i] * cs, a.area[i] * sn};
        const double2 j0 = cmul(ph, xb[2 * i]), j1 = cmul(ph, xb[2 * i + 1]);
        const double2 m0 = cmul(ph, xb[2 * a.P + 2 * i]), m1 = cmul(ph, xb[2 * a.P + 2 * i + 1]);
        const double *t0 = a.tan + 6 * i, *t1 = t0 + 3;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          N[c].x += j0.x * t0[c] + j1.x * t1[c];
          N[c].y += j0.y * t0[c] + j1.y * t1[c];
          M[c].x += m0.x * t0[c] + m1.x * t1[c];
          M[c].y += m0.y * t0[c] + m1.y * t1[c];
        }
      }
      const double th[3] = {w * cp, w * sp, -st}, ph[3] = {-sp, cp, 0.0};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        et.x += N[c].x * th[c] + M[c].x * ph[c];
        et.y += N[c].y * th[c] + M[c].y * ph[c];
        ep.x += N[c].x * ph[c] - M[c].x * th[c];
        ep.y += N[c].y * ph[c] - M[c].y * th[c];
      }
    }
    if (bin >= bins) continue;
    if constexpr (HS == 1) {
      double2* out = a.E + ((long long)r * bins + bin) * 2;
      out[0] = et;
      out[1] = ep;
    } else {
      const double U = et.x * et.x + et.y * et.y + ep.x * ep.x + ep.y * ep.y;
      a.U[((long long)r * 2 + h) * bins + bin] = U;
      const double du = 2.0 * pi / (a.Lu * a.k * a.pitch), dv = 2.0 * pi / (Lv * a.k * a.pitch);
      power += vis ? U * du * dv / sqrt(1.0 - s2) : 0.0;
    }
  }
  if constexpr (HS == 1) return;
  red[threadIdx.x] = power;
  __syncthreads();
  if (threadIdx.x < 64) {   // (fixed order)
    double s = 0.0;
    for (int i = threadIdx.x; i < BIN_THREADS; i += 64) s += red[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (threadIdx.x == 0) a.part[(long long)r * gridDim.x + blockIdx.x] = s;
  }
}

// sum of n values, the same order in every wavefront that forms it
__device__ __forceinline__ double sum_of(const double* __restrict__ v, int n) {
  double s = 0.0;
  for (int i = threadIdx.x & 63; i < n; i += 64) s += v[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  return s;
}

// out[r] = sum of the partial powers of right-hand side r
__global__ void __launch_bounds__(64) power_kernel(const double* __restrict__ part, int parts,
                                                   double* __restrict__ out) {
  const double s = sum_of(part + (long long)blockIdx.x * parts, parts);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// D[r][h][q][p] = 4 pi U / P_rad[r], P_rad[r] the sum of the parts partial
// powers (every workgroup adds those of all right-hand sides, in the same
// order; the first reports them).  D is left alone where a sum is not positive
// and finite, which the call refuses.
constexpr int DIR_THREADS = 256, DIR_RHS = 64;
__global__ void __launch_bounds__(DIR_THREADS) directivity_kernel(const double* __restrict__ part, int parts,
                                                                  int nrhs, const double* __restrict__ U,
                                                                  long long per_rhs, double* __restrict__ D,
                                                                  double* __restrict__ prad) {
  __shared__ double sum[DIR_RHS];
  const int r = blockIdx.y, t = threadIdx.x;
  for (int i = t >> 6; i < nrhs; i += DIR_THREADS / 64) {
    const double s = sum_of(part + (long long)i * parts, parts);
    if ((t & 63) == 0) sum[i] = s;
  }
  __syncthreads();
  if (blockIdx.x == 0 && r == 0 && t < nrhs) prad[t] = sum[t];
  for (int i = 0; i < nrhs; ++i)
    if (!(sum[i] > 0.0) || !isfinite(sum[i])) return;
  const double P = sum[r];
  const double* u = U + r * per_rhs;
  double* d = D + r * per_rhs;
  for (long long i = blockIdx.x * (long long)DIR_THREADS + t; i < per_rhs; i += (long long)gridDim.x * DIR_THREADS)
    d[i] = 4.0 * 3.14159265358979323846 * u[i] / P;
}

int bin_blocks(int Lu, int Lv) { return (int)(((long long)Lu * Lv + BIN_THREADS - 1) / BIN_THREADS); }

// Whether a y pass and single bins take the place of the fused kernel: with few
// columns (p, r) of many bins, whose workgroups leave CUs idle, and with many
// columns of few bins, whose threads outnumber the bins.  HS = 2 (directivity)
// against HS = 1 (far field) as the fused kernel saves two half spaces'
// spectrum reads.  Microseconds fused / by bins, 48 patches, 1 right-hand side:
// HS 2, 64 x 1024 bins 316 / 158, 128 x 1024 321 / 357, 128 x 512 158 / 158, 128 x
// 256 90 / 131, 64 x 64 56 / 102; HS 1, 64 x 1024 295 / 97, 128 x 192 89 / 76, 256
// x 192 96 / 97, 128 x 256 74 / 76, 1024 x 16 90 / 76, 512 x 16 51 / 65.
bool by_bins(int Lu, int Lv, int nrhs, int P, int hs) {
  const int64_t columns = (int64_t)Lu * nrhs;
  if (hs == 2) return (Lv >= 384 && columns <= (Lv < 1024 ? 128 : 64)) || (Lv <= 32 && columns >= std::min(40 * P, 2048));
  return ((Lv >= 192 || Lv == 96) && columns <= 128) || (Lv <= 32 && columns >= std::min(20 * P, 1024));
}

// x pass of the lattice DFT of the unknowns (sign +1) into W[iy][p][r][u]
void lattice_dft_x(int n, int nx, int ny, int nrhs, int Lu, const void* x_dev, void* W, hipStream_t s) {
  const int64_t B = (int64_t)nrhs * n, M = (int64_t)nx * ny;
  FftPass fx;
  fx.L = Lu; fx.n_in = nx; fx.n_out = Lu; fx.batch = n;
  fx.n_lines = nrhs * ny; fx.nl0 = ny;
  fx.in_s1 = M * n; fx.in_s0 = (int64_t)nx * n; fx.in_pt = n;
  fx.out_s1 = n; fx.out_s0 = (int64_t)Lu * B; fx.out_pt = B;
  fx.sign = +1;
  launch_fft_pass(fx, Cx::C128, Cx::C128, Cx::C128, x_dev, W, twiddle_table(Lu, Cx::C128), s);
}

template <int HS> void launch_pattern(int Lv, const PatternArgs& a, hipStream_t s) {
  // the y transform addresses its input with 32-bit offsets
  const int64_t B = (int64_t)a.nrhs * 4 * a.P;
  EMS_CHECK_ARG(Lv * a.Lu * B + B + 1024 < (1LL << 31), "FFT line span exceeds 32-bit offsets");
  const dim3 grid((unsigned)a.Lu, (unsigned)a.nrhs);
  switch (Lv) {
#define EMS_PATTERN(LL)                                                                                 \
  case LL:                                                                                              \
    hipLaunchKernelGGL((pattern_kernel<LL, HS>), grid, dim3((unsigned)Shape<LL, 1>::NT), 0, s, a);      \
    break;
    EMS_PATTERN(2)
    EMS_PATTERN(4)
    EMS_PATTERN(8)
    EMS_PATTERN(16)
    EMS_PATTERN(32)
    EMS_PATTERN(64)
    EMS_PATTERN(128)
    EMS_PATTERN(256)
    EMS_PATTERN(512)
    EMS_PATTERN(1024)
    EMS_PATTERN(24)
    EMS_PATTERN(48)
    EMS_PATTERN(96)
    EMS_PATTERN(192)
    EMS_PATTERN(384)
    EMS_PATTERN(768)
#undef EMS_PATTERN
    default: break;
  }
  EMS_LAUNCH_CHECK();
}

// y pass of a.W into X[q][p][r][u], then the projection by single bins
template <int HS> void launch_bins(int Lv, PatternArgs a, void* X, hipStream_t s) {
  const int64_t B = (int64_t)a.nrhs * 4 * a.P;
  FftPass fy;
  fy.L = Lv; fy.n_in = a.ny; fy.n_out = Lv; fy.batch = (int)B;
  fy.n_lines = a.Lu; fy.nl0 = a.Lu;
  fy.in_s0 = B; fy.in_pt = (int64_t)a.Lu * B;
  fy.out_s0 = B; fy.out_pt = (int64_t)a.Lu * B;
  fy.sign = +1;
  launch_fft_pass(fy, Cx::C128, Cx::C128, Cx::C128, a.W, X, a.tw, s);
  a.W = static_cast<const double2*>(X);
  hipLaunchKernelGGL((bins_kernel<HS>), dim3((unsigned)bin_blocks(a.Lu, Lv), (unsigned)a.nrhs), dim3(BIN_THREADS), 0, s,
                     a, Lv);
  EMS_LAUNCH_CHECK();
}

PatternArgs pattern_args(const GreenGeomDev& g, int ny, int nrhs, int Lu, int Lv, const void* W) {
  PatternArgs a{};
  a.W = static_cast<const double2*>(W);
  a.rho = g.rho;
  a.area = g.area;
  a.tan = g.tan;
  a.tw = static_cast<const double2*>(twiddle_table(Lv, Cx::C128));
  a.P = g.n_patch;
  a.Lu = Lu;
  a.ny = ny;
  a.nrhs = nrhs;
  a.pitch = g.pitch;
  a.k = g.k;
  return a;
}

void check_far_args(const emsurf_geom* geom, int32_t nx, int32_t ny, int32_t nrhs, int32_t Lu, int32_t Lv) {
  EMS_CHECK_ARG(nx >= 1 && ny >= 1 && nx <= 1024 && ny <= 1024, "lattice sizes must be in [1, 1024]");
  EMS_CHECK_ARG(nrhs >= 1 && nrhs <= 64, "nrhs must be in [1, 64]");
  EMS_CHECK_ARG(fft_length_basic(Lu) && fft_length_basic(Lv) && Lu >= nx && Lv >= ny,
                "Lu, Lv must be supported FFT lengths (2^a <= 1024 or 3 * 2^a <= 768) with Lu >= nx, Lv >= ny");
  EMS_CHECK_ARG(geom != nullptr && geom->k > 0, "the far field needs a wavenumber k > 0");
}

}  // namespace
}  // namespace emsurf

using namespace emsurf;

extern "C" emsurf_status emsurf_far_field(const emsurf_geom* geom, int32_t nx, int32_t ny, int32_t nrhs, int32_t Lu,
                                          int32_t Lv, const void* x_dev, void* E_dev, void* stream) {
  try {
    EMS_CHECK_ARG(x_dev != nullptr && E_dev != nullptr, "x_dev and E_dev must be non-NULL");
    check_far_args(geom, nx, ny, nrhs, Lu, Lv);
    hipStream_t s = static_cast<hipStream_t>(stream);
    GreenGeomDev g;
    upload_geom(geom, g, s);
    const size_t b_row = (size_t)nrhs * 4 * g.n_patch * Lu * 16, b_w = Scratch::round(ny * b_row);
    const bool bins = by_bins(Lu, Lv, nrhs, g.n_patch, 1);
    Scratch ws(b_w + (bins ? Lv * b_row : 0));
    void* W = ws.part(b_w);
    lattice_dft_x(4 * g.n_patch, nx, ny, nrhs, Lu, x_dev, W, s);
    PatternArgs a = pattern_args(g, ny, nrhs, Lu, Lv, W);
    a.E = static_cast<double2*>(E_dev);
    if (bins)
      launch_bins<1>(Lv, a, ws.part(Lv * b_row), s);
    else
      launch_pattern<1>(Lv, a, s);
    EMS_HIP(hipStreamSynchronize(s));
    ws.idle();
    g.idle();
    return EMSURF_OK;
  } catch (...) {
    return current_exception_status();
  }
}

extern "C" emsurf_status emsurf_directivity(const emsurf_geom* geom, int32_t nx, int32_t ny, int32_t nrhs, int32_t Lu,
                                            int32_t Lv, const void* x_dev, void* D_dev, double* prad_host,
                                            void* stream) {
  try {
    EMS_CHECK_ARG(x_dev != nullptr && D_dev != nullptr, "x_dev and D_dev must be non-NULL");
    check_far_args(geom, nx, ny, nrhs, Lu, Lv);
    hipStream_t s = static_cast<hipStream_t>(stream);
    GreenGeomDev g;
    upload_geom(geom, g, s);
    const size_t b_row = (size_t)nrhs * 4 * g.n_patch * Lu * 16, b_w = Scratch::round(ny * b_row);
    const bool bins = by_bins(Lu, Lv, nrhs, g.n_patch, 2);
    int parts = bins ? bin_blocks(Lu, Lv) : Lu;
    const long long per_rhs = (long long)2 * Lu * Lv;
    const size_t b_x = bins ? Scratch::round(Lv * b_row) : 0, b_U = Scratch::round(nrhs * per_rhs * 8);
    const size_t b_part = Scratch::round((size_t)nrhs * parts * 8), b_prad = (size_t)nrhs * 8;
    Scratch ws(b_w + b_x + b_U + b_part + 2 * Scratch::round(b_prad));
    void *W = ws.part(b_w), *X = ws.part(b_x);
    double *U = ws.part<double>(b_U), *part = ws.part<double>(b_part);
    double *sums = ws.part<double>(b_prad), *prad = ws.part<double>(b_prad);
    lattice_dft_x(4 * g.n_patch, nx, ny, nrhs, Lu, x_dev, W, s);
    PatternArgs a = pattern_args(g, ny, nrhs, Lu, Lv, W);
    a.U = U;
    a.part = part;
    if (bins)
      launch_bins<2>(Lv, a, X, s);
    else
      launch_pattern<2>(Lv, a, s);
    if (nrhs > 4) {
      // (up to four a workgroup's wavefronts add them at once)
      hipLaunchKernelGGL(power_kernel, dim3((unsigned)nrhs), dim3(64), 0, s, part, parts, sums);
      part = sums;
      parts = 1;
    }
    const long long blocks = (per_rhs + 4 * DIR_THREADS - 1) / (4 * DIR_THREADS);
    hipLaunchKernelGGL(directivity_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096), (unsigned)nrhs),
                       dim3(DIR_THREADS), 0, s, part, parts, nrhs, U, per_rhs, static_cast<double*>(D_dev), prad);
    EMS_LAUNCH_CHECK();
    std::vector<double> pr(nrhs, 0.0);
    EMS_HIP(hipMemcpyAsync(pr.data(), prad, b_prad, hipMemcpyDeviceToHost, s));
    EMS_HIP(hipStreamSynchronize(s));
    ws.idle();
    g.idle();
    for (int r = 0; r < nrhs; ++r)
      EMS_CHECK_ARG(pr[r] > 0 && std::isfinite(pr[r]), "the currents radiate no power (zero or non-finite x)");
    if (prad_host)
      for (int r = 0; r < nrhs; ++r) prad_host[r] = pr[r];
    return EMSURF_OK;
  } catch (...) {
    return current_exception_status();
  }
}
