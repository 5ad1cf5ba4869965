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

// sin of 2*pi*j/16 and, for j = 0..30, of 2*pi*j/120, and what their rounding to
// FP64 leaves out: the constants inside the butterflies of powers of two, and of
// radices 3, 5 and those composed of them (6 to 24, which divide 120)
struct HiLo {
  double hi, lo;
};
__device__ constexpr HiLo sin16(int j) {   // j >= 0
  const double lo[4] = {0.0, -1.0050772696461588e-17, -4.833646656726457e-17, 1.7645047084336677e-17};
  const double v = j % 8 == 4 ? 0.0 : lo[j % 8 < 4 ? j % 8 : 8 - j % 8];
  return {kS16[j % 16], j % 16 < 8 ? v : -v};
}
__device__ constexpr HiLo cos16(int j) { return sin16(j + 4); }
__device__ constexpr HiLo kSin120[31] = {
    {0.0, 0.0}, {0.052335956242943835, -1.9154745404913664e-18}, {0.10452846326765347, 5.525270925166623e-19},
    {0.15643446504023087, 5.047996510305999e-20}, {0.20791169081775934, -5.47375691962595e-18},
    {0.25881904510252074, 2.287249500495561e-17}, {0.30901699437494745, -2.716057601841253e-17},
    {0.35836794954530027, 5.129429438742477e-18}, {0.4067366430758002, -5.150578879759637e-19},
    {0.4539904997395468, -1.2920330362313115e-17}, {0.5, 0.0}, {0.5446390350150271, -2.0392112176790234e-18},
    {0.5877852522924731, -7.93475083819002e-18}, {0.6293203910498375, -4.928960949864041e-17},
    {0.6691306063588582, -2.3743801958426667e-17}, {0.7071067811865476, -4.833646656726457e-17},
    {0.7431448254773942, -9.102893411544583e-18}, {0.7771459614569709, -2.1812891210385366e-17},
    {0.8090169943749475, -2.716057601841253e-17}, {0.838670567945424, -2.0655877157166513e-17},
    {0.8660254037844386, 5.0175421109034514e-17}, {0.8910065241883679, -3.644913950547234e-17},
    {0.9135454576426009, 2.890310230536196e-17}, {0.9335804264972017, 5.99316437034661e-18},
    {0.9510565162951535, 4.0934500900087295e-17}, {0.9659258262890683, -2.5463971562308955e-17},
    {0.9781476007338057, -5.0904377976839195e-17}, {0.9876883405951378, -4.4160180059897935e-17},
    {0.9945218953682733, 4.7061342505091844e-17}, {0.9986295347545738, 4.055160965126569e-17}, {1.0, 0.0}};
__device__ constexpr HiLo sin120(int j) {   // j >= 0
  const HiLo v = kSin120[j % 60 <= 30 ? j % 60 : 60 - j % 60];
  return j % 120 < 60 ? v : HiLo{-v.hi, -v.lo};
}
__device__ constexpr HiLo cos120(int j) { return sin120(j + 30); }

// A constant as the nearest T and the rest.  A constant's rounding is the same
// in every butterfly, so that it adds up over the stages and over forward and
// inverse, where the roundings of products average out.  FP32 structured
// applies of 50 x 50 elements (100 points an axis, two radices 10), error
// against 64 bits: 1.81e-7 with the rounded constants, 1.41e-7 with the rest
// (1.35e-7 at 128 points); 90 x 100 elements 1.80e-7 -> 1.54e-7.  In FP64, 320
// points an axis: 2.56e-16, with radix 16's own rest too 2.17e-16 (2.02e-16 at
// 384 points).  A multiply-add for each, 1.2% of the 90 x 100 apply.
template <typename T> struct Const {
  T hi, lo;
  __device__ constexpr Const(HiLo c)
      : hi(static_cast<T>(c.hi)), lo(static_cast<T>((c.hi - static_cast<double>(static_cast<T>(c.hi))) + c.lo)) {}
};
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
// c x, and c x + d y
template <typename T> __device__ __forceinline__ T times(Const<T> c, T x) { return fmadd(c.hi, x, c.lo * x); }
template <typename T> __device__ __forceinline__ T times2(Const<T> c, T x, Const<T> d, T y) {
  return fmadd(d.hi, y, fmadd(c.hi, x, fmadd(c.lo, x, d.lo * y)));
}
template <typename T> __device__ constexpr Const<T> negated(Const<T> c) {
  c.hi = -c.hi;
  c.lo = -c.lo;
  return c;
}

// v (c + sign i s)
template <typename T, typename V> __device__ __forceinline__ V turn(Const<T> c, Const<T> s, V v, int sign) {
  const Const<T> m = negated(s);
  return V{times2(c, v.x, sign < 0 ? s : m, v.y), times2(c, v.y, sign < 0 ? m : s, v.x)};
}

// factors R = A B of a composite butterfly, 0 for the others
constexpr int composite_a(int R) {
  return R == 6 ? 3 : R == 10 || R == 15 || R == 20 ? 5 : R == 12 ? 4 : R == 24 ? 8 : 0;
}

// In-register DFT of length R: a[k] <- sum_n a[n] e^{sign 2 pi i n k / R}.
// LO: constants with their rest in the powers of two and radix 3 too (the mixed
// lengths), as in the composite radices.
template <int R, typename V, bool LO = false>
__device__ __forceinline__ void dft(V (&a)[R], int sign) {
  using T = typename Real<V>::T;
  if constexpr (R == 1) {
    return;
  } else if constexpr (R == 3) {
    // X1,2 = a0 - (a1 + a2)/2 +- i sign sqrt(3)/2 (a1 - a2)
    constexpr Const<T> s3(sin120(40));
    const V t1 = cadd(a[1], a[2]);
    const V t2 = V{a[0].x - static_cast<T>(0.5) * t1.x, a[0].y - static_cast<T>(0.5) * t1.y};
    const V d = csub(a[1], a[2]);
    const V u = mul_si(LO ? V{times(s3, d.x), times(s3, d.y)} : V{s3.hi * d.x, s3.hi * d.y}, sign);
    a[0] = cadd(a[0], t1);
    a[1] = cadd(t2, u);
    a[2] = csub(t2, u);
  } else if constexpr (R == 5) {
    // real and imaginary rows share the sums a1 +- a4 and a2 +- a3
    constexpr Const<T> c1(cos120(24)), c2(cos120(48)), s1(sin120(24)), s2(sin120(48));
    const V t1 = cadd(a[1], a[4]), t2 = cadd(a[2], a[3]);
    const V d1 = csub(a[1], a[4]), d2 = csub(a[2], a[3]);
    const V m1 = V{a[0].x + times2(c1, t1.x, c2, t2.x), a[0].y + times2(c1, t1.y, c2, t2.y)};
    const V m2 = V{a[0].x + times2(c2, t1.x, c1, t2.x), a[0].y + times2(c2, t1.y, c1, t2.y)};
    const V u1 = mul_si(V{times2(s1, d1.x, s2, d2.x), times2(s1, d1.y, s2, d2.y)}, sign);
    const V u2 = mul_si(V{times2(s2, d1.x, negated(s1), d2.x), times2(s2, d1.y, negated(s1), d2.y)}, sign);
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
      dft<A, V, true>(c[n2], sign);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        if (n2 == 0) continue;
        const int j = n2 * k1 % R * (120 / R);
        c[n2][k1] = turn(Const<T>(cos120(j)), Const<T>(sin120(j)), c[n2][k1], sign);
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      V d[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) d[n2] = c[n2][k1];
      dft<B, V, true>(d, sign);
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
    dft<H, V, LO>(e, sign);
    dft<H, V, LO>(o, sign);
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
        if constexpr (LO) {
          t = turn(Const<T>(cos16(j)), Const<T>(sin16(j)), o[k], sign);
        } else {
          V w{static_cast<T>(kC16[j]), static_cast<T>(sign < 0 ? -kS16[j] : kS16[j])};
          t = cmul(w, o[k]);
        }
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
  static constexpr bool MIXED = false;
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
  static constexpr bool MIXED = true;
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
    dft<R, VC, SH::MIXED>(v[j], a.sign);
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
