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
#include "internal.h"
#include "green.h"

#include <cmath>
#include <mutex>
#include <type_traits>

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

template <int L, int WD, int GEN, int S, int P, typename VI, typename VC, typename VO>
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
    if constexpr (!LAST) __syncthreads();
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
      if constexpr (LAST) {
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
  if constexpr (!LAST) run_stage<L, WD, GEN, S + 1, P * R, VI, VC, VO>(a, lds, in, out, tw, valid, b, g, gg, col, line);
}

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
