// Device pieces of the batched Stockham FFT (fft.hip): register butterflies,
// the stage plan of every length and one stage of a line's transform.  Shared
// by the FFT passes and the radiation pattern's fused y transform.
#pragma once
#include "internal.h"
#include "green.h"

namespace emsurf {
namespace {

template <typename V> struct Real;
template <> struct Real<float2> { using T = float; };
template <> struct Real<double2> { using T = double; };

template <typename V> __device__ __forceinline__ V cmul(V a, V b) {
  return V{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename V> __device__ __forceinline__ V cadd(V a, V b) { return V{a.x + b.x, a.y + b.y}; }
template <typename V> __device__ __forceinline__ V csub(V a, V b) { return V{a.x - b.x, a.y - b.y}; }
// multiply by sign*i
template <typename V> __device__ __forceinline__ V mul_si(V a, int sign) {
  return sign < 0 ? V{a.y, -a.x} : V{-a.y, a.x};
}
template <typename VO, typename VI> __device__ __forceinline__ VO cvt(VI a) {
  using R = typename Real<VO>::T;
  return VO{static_cast<R>(a.x), static_cast<R>(a.y)};
}

// cos and sin of 2*pi*j/16, j = 0..15, correctly rounded FP64 constants
__device__ constexpr double kC16[16] = {
    1.0, 0.92387953251128673848, 0.70710678118654757274, 0.38268343236508978178,
    0.0, -0.38268343236508978178, -0.70710678118654757274, -0.92387953251128673848,
    -1.0, -0.92387953251128673848, -0.70710678118654757274, -0.38268343236508978178,
    0.0, 0.38268343236508978178, 0.70710678118654757274, 0.92387953251128673848};
__device__ constexpr double kS16[16] = {
    0.0, 0.38268343236508978178, 0.70710678118654757274, 0.92387953251128673848,
    1.0, 0.92387953251128673848, 0.70710678118654757274, 0.38268343236508978178,
    0.0, -0.38268343236508978178, -0.70710678118654757274, -0.92387953251128673848,
    -1.0, -0.92387953251128673848, -0.70710678118654757274, -0.38268343236508978178};

// cos and sin of 2*pi*j/120, rounded from extended precision: the twiddles
// inside the composite butterflies (radices 6 to 24 divide 120)
__device__ constexpr double kC120[120] = {
    1.0, 0.9986295347545738, 0.9945218953682733, 0.9876883405951378, 0.9781476007338057, 0.9659258262890683,
    0.9510565162951535, 0.9335804264972017, 0.9135454576426009, 0.8910065241883679, 0.8660254037844386,
    0.838670567945424, 0.8090169943749475, 0.7771459614569709, 0.7431448254773942, 0.7071067811865476,
    0.6691306063588582, 0.6293203910498375, 0.5877852522924731, 0.5446390350150271, 0.5, 0.4539904997395468,
    0.4067366430758002, 0.35836794954530027, 0.30901699437494745, 0.25881904510252074, 0.20791169081775934,
    0.15643446504023087, 0.10452846326765347, 0.052335956242943835, 0.0, -0.052335956242943835,
    -0.10452846326765347, -0.15643446504023087, -0.20791169081775934, -0.25881904510252074, -0.30901699437494745,
    -0.35836794954530027, -0.4067366430758002, -0.4539904997395468, -0.5, -0.5446390350150271, -0.5877852522924731,
    -0.6293203910498375, -0.6691306063588582, -0.7071067811865476, -0.7431448254773942, -0.7771459614569709,
    -0.8090169943749475, -0.838670567945424, -0.8660254037844386, -0.8910065241883679, -0.9135454576426009,
    -0.9335804264972017, -0.9510565162951535, -0.9659258262890683, -0.9781476007338057, -0.9876883405951378,
    -0.9945218953682733, -0.9986295347545738, -1.0, -0.9986295347545738, -0.9945218953682733, -0.9876883405951378,
    -0.9781476007338057, -0.9659258262890683, -0.9510565162951535, -0.9335804264972017, -0.9135454576426009,
    -0.8910065241883679, -0.8660254037844386, -0.838670567945424, -0.8090169943749475, -0.7771459614569709,
    -0.7431448254773942, -0.7071067811865476, -0.6691306063588582, -0.6293203910498375, -0.5877852522924731,
    -0.5446390350150271, -0.5, -0.4539904997395468, -0.4067366430758002, -0.35836794954530027, -0.30901699437494745,
    -0.25881904510252074, -0.20791169081775934, -0.15643446504023087, -0.10452846326765347, -0.052335956242943835,
    0.0, 0.052335956242943835, 0.10452846326765347, 0.15643446504023087, 0.20791169081775934, 0.25881904510252074,
    0.30901699437494745, 0.35836794954530027, 0.4067366430758002, 0.4539904997395468, 0.5, 0.5446390350150271,
    0.5877852522924731, 0.6293203910498375, 0.6691306063588582, 0.7071067811865476, 0.7431448254773942,
    0.7771459614569709, 0.8090169943749475, 0.838670567945424, 0.8660254037844386, 0.8910065241883679,
    0.9135454576426009, 0.9335804264972017, 0.9510565162951535, 0.9659258262890683, 0.9781476007338057,
    0.9876883405951378, 0.9945218953682733, 0.9986295347545738};
__device__ constexpr double kS120[120] = {
    0.0, 0.052335956242943835, 0.10452846326765347, 0.15643446504023087, 0.20791169081775934, 0.25881904510252074,
    0.30901699437494745, 0.35836794954530027, 0.4067366430758002, 0.4539904997395468, 0.5, 0.5446390350150271,
    0.5877852522924731, 0.6293203910498375, 0.6691306063588582, 0.7071067811865476, 0.7431448254773942,
    0.7771459614569709, 0.8090169943749475, 0.838670567945424, 0.8660254037844386, 0.8910065241883679,
    0.9135454576426009, 0.9335804264972017, 0.9510565162951535, 0.9659258262890683, 0.9781476007338057,
    0.9876883405951378, 0.9945218953682733, 0.9986295347545738, 1.0, 0.9986295347545738, 0.9945218953682733,
    0.9876883405951378, 0.9781476007338057, 0.9659258262890683, 0.9510565162951535, 0.9335804264972017,
    0.9135454576426009, 0.8910065241883679, 0.8660254037844386, 0.838670567945424, 0.8090169943749475,
    0.7771459614569709, 0.7431448254773942, 0.7071067811865476, 0.6691306063588582, 0.6293203910498375,
    0.5877852522924731, 0.5446390350150271, 0.5, 0.4539904997395468, 0.4067366430758002, 0.35836794954530027,
    0.30901699437494745, 0.25881904510252074, 0.20791169081775934, 0.15643446504023087, 0.10452846326765347,
    0.052335956242943835, 0.0, -0.052335956242943835, -0.10452846326765347, -0.15643446504023087,
    -0.20791169081775934, -0.25881904510252074, -0.30901699437494745, -0.35836794954530027, -0.4067366430758002,
    -0.4539904997395468, -0.5, -0.5446390350150271, -0.5877852522924731, -0.6293203910498375, -0.6691306063588582,
    -0.7071067811865476, -0.7431448254773942, -0.7771459614569709, -0.8090169943749475, -0.838670567945424,
    -0.8660254037844386, -0.8910065241883679, -0.9135454576426009, -0.9335804264972017, -0.9510565162951535,
    -0.9659258262890683, -0.9781476007338057, -0.9876883405951378, -0.9945218953682733, -0.9986295347545738, -1.0,
    -0.9986295347545738, -0.9945218953682733, -0.9876883405951378, -0.9781476007338057, -0.9659258262890683,
    -0.9510565162951535, -0.9335804264972017, -0.9135454576426009, -0.8910065241883679, -0.8660254037844386,
    -0.838670567945424, -0.8090169943749475, -0.7771459614569709, -0.7431448254773942, -0.7071067811865476,
    -0.6691306063588582, -0.6293203910498375, -0.5877852522924731, -0.5446390350150271, -0.5, -0.4539904997395468,
    -0.4067366430758002, -0.35836794954530027, -0.30901699437494745, -0.25881904510252074, -0.20791169081775934,
    -0.15643446504023087, -0.10452846326765347, -0.052335956242943835};

// factors R = A B of a composite butterfly, 0 for the others
constexpr int composite_a(int R) {
  return R == 6 ? 3 : R == 10 || R == 15 || R == 20 ? 5 : R == 12 ? 4 : R == 24 ? 8 : 0;
}

// In-register DFT of length R: a[k] <- sum_n a[n] e^{sign 2 pi i n k / R}
template <int R, typename V>
__device__ __forceinline__ void dft(V (&a)[R], int sign) {
  using T = typename Real<V>::T;
  if constexpr (R == 1) {
    return;
  } else if constexpr (R == 3) {
    // X1,2 = a0 - (a1 + a2)/2 +- i sign sqrt(3)/2 (a1 - a2)
    const T s3 = static_cast<T>(sign < 0 ? -0.86602540378443864676 : 0.86602540378443864676);
    const V t1 = cadd(a[1], a[2]);
    const V t2 = V{a[0].x - static_cast<T>(0.5) * t1.x, a[0].y - static_cast<T>(0.5) * t1.y};
    const V d = csub(a[1], a[2]);
    const V u = V{-s3 * d.y, s3 * d.x};
    a[0] = cadd(a[0], t1);
    a[1] = cadd(t2, u);
    a[2] = csub(t2, u);
  } else if constexpr (R == 5) {
    // real and imaginary rows share the sums a1 +- a4 and a2 +- a3
    const T c1 = static_cast<T>(kC120[24]), c2 = static_cast<T>(kC120[48]);
    const T s1 = static_cast<T>(kS120[24]), s2 = static_cast<T>(kS120[48]);
    const V t1 = cadd(a[1], a[4]), t2 = cadd(a[2], a[3]);
    const V d1 = csub(a[1], a[4]), d2 = csub(a[2], a[3]);
    const V m1 = V{a[0].x + c1 * t1.x + c2 * t2.x, a[0].y + c1 * t1.y + c2 * t2.y};
    const V m2 = V{a[0].x + c2 * t1.x + c1 * t2.x, a[0].y + c2 * t1.y + c1 * t2.y};
    const V u1 = mul_si(V{s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y}, sign);
    const V u2 = mul_si(V{s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y}, sign);
    a[0] = V{a[0].x + t1.x + t2.x, a[0].y + t1.y + t2.y};
    a[1] = cadd(m1, u1);
    a[4] = csub(m1, u1);
    a[2] = cadd(m2, u2);
    a[3] = csub(m2, u2);
  } else if constexpr (composite_a(R) > 0) {
    // n = B n1 + n2, k = k1 + A k2: B butterflies of length A, twiddles, A of length B
    constexpr int A = composite_a(R), B = R / A;
    V c[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) c[n2][n1] = a[B * n1 + n2];
      dft<A, V>(c[n2], sign);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        if (n2 == 0) continue;
        const int j = n2 * k1 % R * (120 / R);
        c[n2][k1] = cmul(V{static_cast<T>(kC120[j]), static_cast<T>(sign < 0 ? -kS120[j] : kS120[j])}, c[n2][k1]);
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      V d[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) d[n2] = c[n2][k1];
      dft<B, V>(d, sign);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) a[k1 + A * k2] = d[k2];
    }
  } else if constexpr (R == 2) {
    V t = a[0];
    a[0] = cadd(t, a[1]);
    a[1] = csub(t, a[1]);
  } else {
    constexpr int H = R / 2;
    V e[H], o[H];
#pragma unroll
    for (int i = 0; i < H; ++i) { e[i] = a[2 * i]; o[i] = a[2 * i + 1]; }
    dft<H, V>(e, sign);
    dft<H, V>(o, sign);
#pragma unroll
    for (int k = 0; k < H; ++k) {
      constexpr int step = 16 / R;
      const int j = k * step;  // angle 2 pi j / 16
      V t;
      if (j == 0) {
        t = o[k];
      } else if (j == 4) {
        t = mul_si(o[k], sign);
      } else {
        V w{static_cast<T>(kC16[j]), static_cast<T>(sign < 0 ? -kS16[j] : kS16[j])};
        t = cmul(w, o[k]);
      }
      a[k] = cadd(e[k], t);
      a[k + H] = csub(e[k], t);
    }
  }
}

// Inputs generated in the first stage instead of loaded: the point-sampled
// coupling entries of kernel columns c0 + col (column c = vp n + u, v from vp
// in the pair_fill_v order when vperm) at lattice slot (point, line) of the x
// pass of the kernel transform.
struct GreenGen {
  const double* rho = nullptr;
  const double* area = nullptr;
  const double* tan = nullptr;
  int P = 0, nx = 0, ny = 0, Ly = 0, c0 = 0, n = 0, vperm = 0;   // rows in the green_fill_u order
  double pitch = 0, k = 0;
};

struct PassArgs {
  int n_in, n_out, batch, nl0;
  long long in_s0, in_s1, out_s0, out_s1;
  int in_pt, out_pt;   // point strides (elements); host checks they fit 32 bits
  int sign;
  double scale;
};

// Compile-time plan of a transform length: radix of each stage, G threads per
// column and BT columns per workgroup (NT = G BT threads).  A stage's L / R
// butterflies go round the G threads (the last round partly idle where G does
// not divide them).  WD = 2 doubles the threads and so the columns per
// workgroup (256-byte runs per point in FP32; 64 KB of LDS at L = 256).
//
// Lengths 2^a (2..1024) and 3 * 2^a (24..768) run radix-16 or radix-8 stages
// while possible, then what is left of the power of two, then radix 3.
template <int L, int WD = 1> struct Shape {
  static constexpr bool R3 = L % 3 == 0;
  static constexpr int VPT = R3 ? 24 : (L >= 16 ? 16 : L);
  static constexpr int NT = (R3 ? 128 : 256) * WD;
  static constexpr int G = L / VPT;
  static constexpr int BT = NT / G;
  static constexpr int nst() {
    int n = 0;
    if (R3) {
      int r = L / 3;
      while (r >= 8) { r /= 8; ++n; }
      return n + (r > 1 ? 1 : 0) + 1;
    }
    int r = L;
    while (r >= 16) { r /= 16; ++n; }
    return n + (r > 1 ? 1 : 0);
  }
  static constexpr int radix(int s) {
    if (R3) {
      int r = L / 3;
      for (int i = 0; i < s; ++i) {
        if (r == 1) return 3;
        r /= (r >= 8 ? 8 : r);
      }
      return r == 1 ? 3 : (r >= 8 ? 8 : r);
    }
    int r = L;
    for (int i = 0; i < s; ++i) r /= (r >= 16 ? 16 : r);
    return r >= 16 ? 16 : r;
  }
  static constexpr int NST = nst();
};

// The lengths between them, products of 2, 3 and 5: one or two stages of
// composite radices (one LDS exchange), with 16 or 32 columns and 10 to 24
// values per thread.
template <int L_, int WD, int G_, int BT_, int R0, int R1, int R2> struct MixedShape {
  static constexpr int G = G_, BT = BT_ * WD, NT = G * BT;
  static constexpr int NST = R2 > 1 ? 3 : R1 > 1 ? 2 : 1;
  static constexpr int radix(int s) { return s == 0 ? R0 : s == 1 ? R1 : R2; }
  static_assert(R0 * R1 * R2 == L_, "radices multiply to the length");
};
// length, threads per column, columns per workgroup, radices
#define EMS_MIXED_LENGTHS(X)                                                                             \
  X(6, 1, 64, 6, 1, 1) X(10, 1, 64, 10, 1, 1) X(12, 1, 64, 12, 1, 1) X(20, 1, 64, 20, 1, 1)              \
  X(36, 6, 32, 6, 6, 1) X(40, 4, 32, 10, 4, 1) X(60, 4, 32, 15, 4, 1) X(72, 6, 32, 12, 6, 1)             \
  X(80, 4, 32, 20, 4, 1) X(100, 10, 16, 10, 10, 1) X(120, 8, 16, 15, 8, 1) X(144, 12, 16, 12, 12, 1)     \
  X(160, 8, 16, 20, 8, 1) X(180, 12, 16, 15, 12, 1) X(200, 10, 16, 20, 10, 1) X(225, 15, 16, 15, 15, 1)  \
  X(240, 16, 16, 16, 15, 1) X(288, 12, 16, 24, 12, 1) X(320, 16, 8, 8, 8, 5) X(360, 24, 8, 24, 15, 1)    \
  X(400, 20, 8, 20, 20, 1) X(480, 24, 8, 24, 20, 1) X(576, 24, 8, 24, 24, 1)
#define EMS_MIXED_SHAPE(L, G, BT, R0, R1, R2) \
  template <int WD> struct Shape<L, WD> : MixedShape<L, WD, G, BT, R0, R1, R2> {};
EMS_MIXED_LENGTHS(EMS_MIXED_SHAPE)
#undef EMS_MIXED_SHAPE

// Column b of a transform left in LDS (TOLDS below) at point pos: the columns
// of a point are permuted by its index, so that lanes on consecutive points of
// one column meet different banks.
template <int L, int WD> __device__ __forceinline__ int lds_column(int pos, int b) {
  constexpr int BT = Shape<L, WD>::BT;
  return pos * BT + (b ^ (pos & (BT < 16 ? BT - 1 : 15)));
}

// Stage S and those after it.  TOLDS: the transform ends in lds (whose L BT
// values every stage uses) at lds_column instead of in `out`.
template <int L, int WD, int GEN, int S, int P, typename VI, typename VC, typename VO, bool TOLDS = false>
__device__ __forceinline__ void run_stage(const PassArgs& a, VC* lds, const VI* __restrict__ in,
                                          VO* __restrict__ out, const VC* __restrict__ tw, bool valid, int b,
                                          int g, const GreenGen& gg, int col, int line) {
  using SH = Shape<L, WD>;
  constexpr int R = SH::radix(S);
  constexpr int LR = L / R;
  constexpr int G = SH::G;
  constexpr int NB = (LR + G - 1) / G;
  constexpr bool EVEN = LR % G == 0;   // every thread has NB butterflies
  constexpr int BT = SH::BT;
  constexpr bool FIRST = S == 0;
  constexpr bool LAST = S == SH::NST - 1;
  VC v[NB][R];
  // ---- load
  if constexpr (FIRST && GEN) {
    // this thread's kernel column (u, v) and the line's lattice offset dy
    bool oky;
    const int dy = slot_to_offset(line, gg.Ly, gg.ny, &oky);
    const int c = gg.c0 + col;
    const int vp = c / gg.n;
    const int u = green_fill_u(c - vp * gg.n, gg.P);
    const int vv = gg.vperm ? pair_fill_v(vp, gg.n) : vp;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i = g + G * j;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int pos = i + q * LR;
        bool okx = false;
        const int dx = slot_to_offset(pos, L, gg.nx, &okx);
        if (valid && oky && okx && pos < a.n_in && (EVEN || i < LR))
          v[j][q] = cvt<VC>(green_entry(gg.rho, gg.area, gg.tan, gg.P, gg.pitch, gg.k, dx, dy, u, vv));
        else
          v[j][q] = VC{0, 0};
      }
    }
  } else if constexpr (FIRST) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i = g + G * j;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int pos = i + q * LR;
        if (valid && pos < a.n_in && (EVEN || i < LR))
          v[j][q] = cvt<VC>(in[(unsigned)(pos * a.in_pt)]);
        else
          v[j][q] = VC{0, 0};
      }
    }
  } else {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i = g + G * j;
#pragma unroll
      for (int q = 0; q < R; ++q) v[j][q] = EVEN || i < LR ? lds[(i + q * LR) * BT + b] : VC{0, 0};
    }
    if constexpr (!LAST || TOLDS) __syncthreads();
  }
  // ---- twiddle + butterfly
  constexpr int TSTR = L / (P * R);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if constexpr (!FIRST) {
      const int i = g + G * j;
      const int k = i % P;
#pragma unroll
      for (int q = 1; q < R; ++q) {
        VC w = tw[q * k * TSTR];   // q k L / (P R) < L
        if (a.sign > 0) w.y = -w.y;
        v[j][q] = cmul(v[j][q], w);
      }
    }
    dft<R, VC>(v[j], a.sign);
  }
  // ---- store
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i = g + G * j;
    if (!EVEN && i >= LR) continue;
    const int k = i % P;
    const int base = (i - k) * R + k;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int pos = base + q * P;
      if constexpr (LAST && TOLDS) {
        lds[lds_column<L, WD>(pos, b)] = v[j][q];
      } else if constexpr (LAST) {
        if (valid && pos < a.n_out) {
          VC r = v[j][q];
          using T = typename Real<VC>::T;
          if (a.scale != 1.0) {
            const T sc = static_cast<T>(a.scale);
            r.x *= sc;
            r.y *= sc;
          }
          out[(unsigned)(pos * a.out_pt)] = cvt<VO>(r);
        }
      } else {
        lds[pos * BT + b] = v[j][q];
      }
    }
  }
  if constexpr (!LAST)
    run_stage<L, WD, GEN, S + 1, P * R, VI, VC, VO, TOLDS>(a, lds, in, out, tw, valid, b, g, gg, col, line);
}

}  // namespace
}  // namespace emsurf
