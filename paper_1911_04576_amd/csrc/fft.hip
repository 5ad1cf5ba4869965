// Batched Stockham FFT along one lattice axis, for the circulant-embedded
// coupling product of Sec. IV-B (eq. (LJV5) and its 2-D generalisation).
//
// Layout: every transform point holds a contiguous run of batch columns
// (local unknowns u, or (rhs, u) pairs, or (v, u) kernel entries), so a
// workgroup owns BT consecutive columns of one line and all L points of the
// line; global loads and stores are coalesced along the batch.  The first
// radix stage reads global memory directly (skipping the zero padding:
// points >= n_in are never loaded), intermediate stages exchange through LDS
// in place, and the last stage writes global memory directly, dropping the
// points >= n_out (the crop of the inverse transform).
//
// G threads share a column; radices 2 to 24 run as register butterflies.  The
// arithmetic type may differ from the input and output types (FP64 <-> FP32
// converting loads and stores for the mixed-precision solve).
#include "fft_device.h"

#include <cmath>
#include <mutex>
#include <type_traits>

namespace emsurf {
namespace {

template <int L, int WD, int GEN, typename VI, typename VC, typename VO>
__global__ void __launch_bounds__((Shape<L, WD>::NT))
    fft_pass_kernel(PassArgs a, const VI* __restrict__ in, VO* __restrict__ out, const VC* __restrict__ tw,
                    GreenGen gg) {
  using SH = Shape<L, WD>;
  __shared__ VC lds[SH::NST > 1 ? L * SH::BT : 1];
  const int t = threadIdx.x;
  const int b = t % SH::BT;
  const int g = t / SH::BT;
  const long long line = blockIdx.y;
  const long long l1 = line / a.nl0, l0 = line - l1 * a.nl0;
  const int col = blockIdx.x * SH::BT + b;
  const bool valid = col < a.batch;
  // uniform line bases, per-thread 32-bit offsets
  const VI* inl = in + (l1 * a.in_s1 + l0 * a.in_s0 + (long long)blockIdx.x * SH::BT) + b;
  VO* outl = out + (l1 * a.out_s1 + l0 * a.out_s0 + (long long)blockIdx.x * SH::BT) + b;
  run_stage<L, WD, GEN, 0, 1, VI, VC, VO>(a, lds, inl, outl, tw, valid, b, g, gg, col, (int)l0);
}

template <int L, int WD, typename VI, typename VC, typename VO, int GEN = 0>
void launch_L(const PassArgs& a, int batch, unsigned lines, const void* in, void* out, const void* tw, hipStream_t s,
              const GreenGen& gg = GreenGen{}) {
  const unsigned tiles = (unsigned)((batch + Shape<L, WD>::BT - 1) / Shape<L, WD>::BT);
  hipLaunchKernelGGL((fft_pass_kernel<L, WD, GEN, VI, VC, VO>), dim3(tiles, lines), dim3(Shape<L, WD>::NT), 0, s, a,
                     static_cast<const VI*>(in), static_cast<VO*>(out), static_cast<const VC*>(tw), gg);
}

constexpr bool mixed_length(int L) {
#define EMS_IS_LENGTH(LL, ...) L == LL ||
  return EMS_MIXED_LENGTHS(EMS_IS_LENGTH) false;
#undef EMS_IS_LENGTH
}

constexpr bool wide_length(int L) { return L == 64 || L == 128 || L == 256 || (L >= 100 && mixed_length(L)); }

template <typename VI, typename VC, typename VO>
void launch_typed(int L, const PassArgs& a, int batch, unsigned lines, const void* in, void* out, const void* tw,
                  hipStream_t s) {
  // FP32 arithmetic at power-of-two lengths 64..256 with at least 64 columns
  // takes the doubled workgroup (measured 5-7% faster at L = 256 with 192 and
  // 768 columns), and so do the mixed lengths from 100 on, whose runs are 128
  // bytes otherwise; FP64 keeps 256 threads, whose LDS would double to 128 KB
  constexpr bool f32 = std::is_same<VC, float2>::value;
  const bool wide = f32 && batch >= 64;
#define EMS_FFT_CASE(LL)                                                           \
  case LL: {                                                                       \
    if constexpr (f32 && wide_length(LL)) {                                        \
      if (wide) {                                                                  \
        launch_L<LL, 2, VI, VC, VO>(a, batch, lines, in, out, tw, s);              \
        break;                                                                     \
      }                                                                            \
    }                                                                              \
    launch_L<LL, 1, VI, VC, VO>(a, batch, lines, in, out, tw, s);                  \
    break;                                                                         \
  }
#define EMS_FFT_MIXED(LL, ...) EMS_FFT_CASE(LL)
  switch (L) {
    EMS_FFT_CASE(2)
    EMS_FFT_CASE(4)
    EMS_FFT_CASE(8)
    EMS_FFT_CASE(16)
    EMS_FFT_CASE(32)
    EMS_FFT_CASE(64)
    EMS_FFT_CASE(128)
    EMS_FFT_CASE(256)
    EMS_FFT_CASE(512)
    EMS_FFT_CASE(1024)
    EMS_FFT_CASE(24)
    EMS_FFT_CASE(48)
    EMS_FFT_CASE(96)
    EMS_FFT_CASE(192)
    EMS_FFT_CASE(384)
    EMS_FFT_CASE(768)
    EMS_MIXED_LENGTHS(EMS_FFT_MIXED)
    default: break;
  }
#undef EMS_FFT_MIXED
#undef EMS_FFT_CASE
}


// ----------------------------------------------------------------------------- small lattices
// Both axes of the padded transform in one launch, by plain sums: with up to
// 16 points per axis a pass is launch and latency.  A workgroup owns 16
// columns and S x frequencies (forward) or S x elements (inverse), so that the
// sums along x of every row and then those along y stay inside it; the x sums
// read memory once for the S, the y sums LDS.  Every output is the same
// sequence of multiply-adds whatever S, which follows the column count: 1
// leaves a few columns the most workgroups, 4 reads the least.  Sums run in
// FP64 in both precisions (they are not what bounds the kernel).  T-apply of
// 4 x 4 elements, n_eq 96, 1 RHS, FP64: 19.4 -> 12.6 us with the split block
// product.
constexpr int SM_COLS = 16, SM_ROWS = 16;

__device__ __forceinline__ void cfma_d(double2& a, double2 x, double2 w) {
  a.x = __builtin_fma(-x.y, w.y, __builtin_fma(x.x, w.x, a.x));
  a.y = __builtin_fma(x.y, w.x, __builtin_fma(x.x, w.y, a.y));
}

// W[j] = exp(-+ 2 pi i j / L) in LDS (minus for sign < 0)
__device__ __forceinline__ void load_twiddles(double2* w, const double2* __restrict__ tw, int L, int sign) {
  for (int j = threadIdx.x; j < L; j += blockDim.x) {
    const double2 v = tw[j];
    w[j] = double2{v.x, sign < 0 ? v.y : -v.y};
  }
}

// step of a twiddle index: k i mod L for i = 0, 1, .. (k < L)
__device__ __forceinline__ int next_index(int idx, int k, int L) {
  idx += k;
  return idx >= L ? idx - L : idx;
}

// x[r][iy][ix][u] -> X[ky][kx][r][u]; grid (column tiles, Lx / S up)
template <int S, typename VI, typename VO>
__global__ void __launch_bounds__(SM_COLS * SM_ROWS)
    small_forward_kernel(const VI* __restrict__ x, VO* __restrict__ X, const double2* __restrict__ twx,
                         const double2* __restrict__ twy, int nx, int ny, int Lx, int Ly, int n, int B) {
  __shared__ double2 wx[16], wy[16], rows[S][16][SM_COLS];
  const int b = threadIdx.x % SM_COLS, row = threadIdx.x / SM_COLS, k0 = blockIdx.y * S;
  const int col = blockIdx.x * SM_COLS + b, r = col / n, u = col - r * n;
  load_twiddles(wx, twx, Lx, -1);
  load_twiddles(wy, twy, Ly, -1);
  __syncthreads();
  if (row < ny && col < B) {
    const VI* xr = x + ((long long)r * ny + row) * nx * n + u;
    double2 acc[S] = {};
    int idx[S] = {};
#pragma unroll 4
    for (int i = 0; i < nx; ++i) {
      const double2 v = cvt<double2>(xr[i * n]);
#pragma unroll
      for (int j = 0; j < S; ++j) {
        cfma_d(acc[j], v, wx[idx[j]]);
        idx[j] = next_index(idx[j], k0 + j < Lx ? k0 + j : 0, Lx);
      }
    }
#pragma unroll
    for (int j = 0; j < S; ++j) rows[j][row][b] = acc[j];
  }
  __syncthreads();
  if (row < Ly && col < B) {
    double2 acc[S] = {};
    for (int i = 0, idx = 0; i < ny; ++i, idx = next_index(idx, row, Ly)) {
      const double2 w = wy[idx];
#pragma unroll
      for (int j = 0; j < S; ++j) cfma_d(acc[j], rows[j][i][b], w);
    }
#pragma unroll
    for (int j = 0; j < S; ++j)
      if (k0 + j < Lx) X[((long long)row * Lx + k0 + j) * B + col] = cvt<VO>(acc[j]);
  }
}

// Y[ky][kx][r][u] -> y[r][iy][ix][u] / (Lx Ly); grid (column tiles, nx / S up)
template <int S, typename VI, typename VO>
__global__ void __launch_bounds__(SM_COLS * SM_ROWS)
    small_inverse_kernel(const VI* __restrict__ Y, VO* __restrict__ y, const double2* __restrict__ twx,
                         const double2* __restrict__ twy, int nx, int ny, int Lx, int Ly, int n, int B) {
  __shared__ double2 wx[16], wy[16], rows[S][16][SM_COLS];
  const int b = threadIdx.x % SM_COLS, row = threadIdx.x / SM_COLS, i0 = blockIdx.y * S;
  const int col = blockIdx.x * SM_COLS + b, r = col / n, u = col - r * n;
  load_twiddles(wx, twx, Lx, +1);
  load_twiddles(wy, twy, Ly, +1);
  __syncthreads();
  if (row < Ly && col < B) {
    const VI* Yr = Y + (long long)row * Lx * B + col;
    double2 acc[S] = {};
    int idx[S] = {};
#pragma unroll 4
    for (int k = 0; k < Lx; ++k) {
      const double2 v = cvt<double2>(Yr[(long long)k * B]);
#pragma unroll
      for (int j = 0; j < S; ++j) {
        cfma_d(acc[j], v, wx[idx[j]]);
        idx[j] = next_index(idx[j], i0 + j < nx ? i0 + j : 0, Lx);
      }
    }
#pragma unroll
    for (int j = 0; j < S; ++j) rows[j][row][b] = acc[j];
  }
  __syncthreads();
  if (row < ny && col < B) {
    double2 acc[S] = {};
    for (int k = 0, idx = 0; k < Ly; ++k, idx = next_index(idx, row, Ly)) {
      const double2 w = wy[idx];
#pragma unroll
      for (int j = 0; j < S; ++j) cfma_d(acc[j], rows[j][k][b], w);
    }
    const double f = 1.0 / ((double)Lx * (double)Ly);
    VO* yr = y + ((long long)r * ny + row) * nx * n + u;
#pragma unroll
    for (int j = 0; j < S; ++j)
      if (i0 + j < nx) yr[(long long)(i0 + j) * n] = cvt<VO>(double2{acc[j].x * f, acc[j].y * f});
  }
}

template <int S, typename VI, typename VO>
void launch_small_s(const SmallDft& d, const void* in, void* out, hipStream_t s) {
  const double2* twx = static_cast<const double2*>(twiddle_table(d.Lx, Cx::C128));
  const double2* twy = static_cast<const double2*>(twiddle_table(d.Ly, Cx::C128));
  const int B = d.nrhs * d.n, outs = d.sign < 0 ? d.Lx : d.nx;
  const dim3 grid((unsigned)((B + SM_COLS - 1) / SM_COLS), (unsigned)((outs + S - 1) / S));
  if (d.sign < 0)
    hipLaunchKernelGGL((small_forward_kernel<S, VI, VO>), grid, dim3(SM_COLS * SM_ROWS), 0, s,
                       static_cast<const VI*>(in), static_cast<VO*>(out), twx, twy, d.nx, d.ny, d.Lx, d.Ly, d.n, B);
  else
    hipLaunchKernelGGL((small_inverse_kernel<S, VI, VO>), grid, dim3(SM_COLS * SM_ROWS), 0, s,
                       static_cast<const VI*>(in), static_cast<VO*>(out), twx, twy, d.nx, d.ny, d.Lx, d.Ly, d.n, B);
}

template <typename VI, typename VO>
void launch_small(const SmallDft& d, const void* in, void* out, hipStream_t s) {
  const int B = d.nrhs * d.n, outs = d.sign < 0 ? d.Lx : d.nx;
  if ((int64_t)(B + SM_COLS - 1) / SM_COLS * outs >= 1024)
    launch_small_s<4, VI, VO>(d, in, out, s);
  else
    launch_small_s<1, VI, VO>(d, in, out, s);
}

std::mutex g_tw_mu;
std::map<std::pair<int, int>, DevBuf*> g_tw;

}  // namespace

const void* twiddle_lookup(int L, Cx t) {
  int dev = 0;
  EMS_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_tw_mu);
  auto it = g_tw.find({L, (t == Cx::C128 ? 1 : 0) + 2 * dev});
  return it == g_tw.end() ? nullptr : it->second->p;
}

const void* twiddle_table(int L, Cx t) {
  int dev = 0;
  EMS_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_tw_mu);
  const int key_t = (t == Cx::C128 ? 1 : 0) + 2 * dev;
  auto it = g_tw.find({L, key_t});
  if (it != g_tw.end()) return it->second->p;
  std::vector<double> h64(2 * (size_t)L);
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int j = 0; j < L; ++j) {
    // exact symmetry reduction keeps every entry correctly rounded to FP64
    const long double ang = -2.0L * pi * (long double)j / (long double)L;
    h64[2 * j] = (double)cosl(ang);
    h64[2 * j + 1] = (double)sinl(ang);
  }
  DevBuf* buf = new DevBuf();
  if (t == Cx::C128) {
    buf->alloc(h64.size() * sizeof(double));
    EMS_HIP(hipMemcpy(buf->p, h64.data(), buf->bytes, hipMemcpyHostToDevice));
  } else {
    std::vector<float> h32(h64.size());
    for (size_t i = 0; i < h64.size(); ++i) h32[i] = (float)h64[i];
    buf->alloc(h32.size() * sizeof(float));
    EMS_HIP(hipMemcpy(buf->p, h32.data(), buf->bytes, hipMemcpyHostToDevice));
  }
  g_tw[{L, key_t}] = buf;
  return buf->p;
}

bool fft_length_basic(int L) {
  if (L >= 2 && L <= 1024 && (L & (L - 1)) == 0) return true;
  if (L % 3 != 0) return false;
  const int q = L / 3;
  return q >= 8 && q <= 256 && (q & (q - 1)) == 0;
}

int fft_length_basic_at_least(int v) {
  int best = 2;
  while (best < v) best <<= 1;
  for (int q = 8; 3 * q <= 768; q <<= 1)
    if (3 * q >= v && 3 * q < best) best = 3 * q;
  return best;
}

// The padded spectrum holds Lx Ly blocks, and streaming them is most of an
// apply, so a lattice takes the shortest length that holds it: 90 x 100
// elements pad to 180 x 200 frequencies, where 192 x 256 took 37% more (FP32
// structured T-apply with 4 RHS at n_eq 192: 1.10 -> 0.85 ms; FP64 A-apply of
// 23 x 17 elements of 150 unknowns with 6 RHS, 48 x 48 -> 48 x 36: 245 -> 185 us).
int fft_length_at_least(int v) {
  int best = fft_length_basic_at_least(v);
  for (int L = v; L < best; ++L)
    if (mixed_length(L)) best = L;
  return best;
}

namespace {
PassArgs pass_args(const FftPass& p) {
  EMS_CHECK_ARG(fft_length_basic(p.L) || mixed_length(p.L), "internal: no FFT kernel of this length");
  EMS_CHECK_ARG(p.n_in >= 1 && p.n_in <= p.L && p.n_out >= 1 && p.n_out <= p.L, "FFT prune/crop sizes out of range");
  EMS_CHECK_ARG(p.batch >= 1 && p.n_lines >= 1 && p.nl0 >= 1, "FFT batch/lines must be positive");
  EMS_CHECK_ARG(p.n_lines <= 65535, "FFT pass has more than 65535 lines");
  const long long span_in = (long long)p.L * p.in_pt + p.batch + 1024;
  const long long span_out = (long long)p.L * p.out_pt + p.batch + 1024;
  EMS_CHECK_ARG(span_in < (1LL << 31) && span_out < (1LL << 31), "FFT line span exceeds 32-bit offsets");
  PassArgs a{};
  a.n_in = p.n_in;
  a.n_out = p.n_out;
  a.batch = p.batch;
  a.nl0 = p.nl0;
  a.in_s0 = p.in_s0; a.in_s1 = p.in_s1; a.out_s0 = p.out_s0; a.out_s1 = p.out_s1;
  a.in_pt = (int)p.in_pt; a.out_pt = (int)p.out_pt;
  a.sign = p.sign;
  a.scale = p.scale;
  return a;
}
}  // namespace

void launch_fft_pass_green(const FftPass& p, const GreenGeomDev& geo, int nx, int ny, int Ly, int64_t c0, int n,
                           int vperm, void* out, const void* twiddles, hipStream_t s) {
  const PassArgs a = pass_args(p);
  // the twiddle table stands in for the input pointer, which the generating
  // first stage never reads
  EMS_CHECK_ARG(p.nl0 == p.n_lines && p.n_lines == Ly && n == 4 * geo.n_patch && c0 >= 0 &&
                    c0 + p.batch <= (int64_t)n * n,
                "internal: generating kernel pass shape");
  GreenGen gg;
  gg.rho = geo.rho;
  gg.area = geo.area;
  gg.tan = geo.tan;
  gg.P = geo.n_patch;
  gg.nx = nx;
  gg.ny = ny;
  gg.Ly = Ly;
  gg.c0 = (int)c0;
  gg.n = n;
  gg.vperm = vperm;
  gg.pitch = geo.pitch;
  gg.k = geo.k;
  const unsigned lines = (unsigned)p.n_lines;
#define EMS_FFT_GEN(LL)                                                                           \
  case LL:                                                                                        \
    launch_L<LL, 1, double2, double2, double2, 1>(a, p.batch, lines, twiddles, out, twiddles, s, gg); \
    break;
  switch (p.L) {
    EMS_FFT_GEN(2)
    EMS_FFT_GEN(4)
    EMS_FFT_GEN(8)
    EMS_FFT_GEN(16)
    EMS_FFT_GEN(32)
    EMS_FFT_GEN(64)
    EMS_FFT_GEN(128)
    EMS_FFT_GEN(256)
    EMS_FFT_GEN(512)
    EMS_FFT_GEN(1024)
    EMS_FFT_GEN(24)
    EMS_FFT_GEN(48)
    EMS_FFT_GEN(96)
    EMS_FFT_GEN(192)
    EMS_FFT_GEN(384)
    EMS_FFT_GEN(768)
#define EMS_FFT_GEN_MIXED(LL, ...) EMS_FFT_GEN(LL)
    EMS_MIXED_LENGTHS(EMS_FFT_GEN_MIXED)
#undef EMS_FFT_GEN_MIXED
    default: break;
  }
#undef EMS_FFT_GEN
  EMS_LAUNCH_CHECK();
}

// Up to 16 points an axis and 128 in all.  A rule on the lattice alone, so that
// a right-hand side's bits do not depend on how many share the apply: T-applies
// of 5 x 5 and 4 x 8 elements took 0.77 to 1.01 of the separate passes' time
// over 1 .. 32 RHS and n_eq 96 .. 288, of 8 x 8 elements (256 points) 0.75 to
// 0.95 with up to 4 RHS but 1.02 to 1.07 from 12 RHS.
bool small_dft_fits(int Lx, int Ly) { return Lx <= 16 && Ly <= 16 && Lx * Ly <= 128; }

void launch_small_dft(const SmallDft& d, Cx tin, Cx tout, const void* in, void* out, hipStream_t s) {
  EMS_CHECK_ARG(small_dft_fits(d.Lx, d.Ly) && d.nx <= d.Lx && d.ny <= d.Ly && d.nx >= 1 && d.ny >= 1 && d.n >= 1 &&
                    d.nrhs >= 1,
                "internal: small transform sizes");
  if (tin == Cx::C128 && tout == Cx::C128) launch_small<double2, double2>(d, in, out, s);
  else if (tin == Cx::C128) launch_small<double2, float2>(d, in, out, s);
  else if (tout == Cx::C128) launch_small<float2, double2>(d, in, out, s);
  else launch_small<float2, float2>(d, in, out, s);
  EMS_LAUNCH_CHECK();
}

void launch_fft_pass(const FftPass& p, Cx tin, Cx tcomp, Cx tout, const void* in, void* out,
                     const void* twiddles, hipStream_t s) {
  const PassArgs a = pass_args(p);
  const unsigned lines = (unsigned)p.n_lines;
  if (tcomp == Cx::C128) {
    EMS_CHECK_ARG(tin == Cx::C128 && tout == Cx::C128, "FP64 FFT needs FP64 input and output");
    launch_typed<double2, double2, double2>(p.L, a, p.batch, lines, in, out, twiddles, s);
  } else {
    if (tin == Cx::C128 && tout == Cx::C64)
      launch_typed<double2, float2, float2>(p.L, a, p.batch, lines, in, out, twiddles, s);
    else if (tin == Cx::C64 && tout == Cx::C128)
      launch_typed<float2, float2, double2>(p.L, a, p.batch, lines, in, out, twiddles, s);
    else if (tin == Cx::C64 && tout == Cx::C64)
      launch_typed<float2, float2, float2>(p.L, a, p.batch, lines, in, out, twiddles, s);
    else
      launch_typed<double2, float2, double2>(p.L, a, p.batch, lines, in, out, twiddles, s);
  }
  EMS_LAUNCH_CHECK();
}

}  // namespace emsurf
