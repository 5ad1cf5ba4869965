// FP64 vector kernels of the batched GMRES solves (Sec. IV-A): Gram-Schmidt
// against the Arnoldi basis, norms, residuals and the solution update
// x += V y.  Vectors are c128, N values each.  Reductions are two-stage and
// atomic-free (per-workgroup partial sums, added in a fixed order), and a
// vector's split over workgroups depends on N alone, so results are bitwise
// reproducible and never depend on the other vectors of a launch.
//
// One Arnoldi step (classical Gram-Schmidt twice) is four kernels that each
// end in partial sums or begin by adding up those of the kernel before:
//   dots       c1 = V^H w, ||w||^2                      reads V and w
//   update     w' = w - V c1, then c2 = V^H w'          reads V and w, writes w'
//   update     w'' = w' - V c2, then ||w''||^2          reads V and w', writes w''
//   normalise  w'' / ||w''||                            reads and writes w''
// The coefficients and norms go straight to host memory, and the scaling
// needs no answer from the host.  Bound by memory, and on small surfaces by
// launches: as separate dot, reduce, update, copy and scale launches a step
// took 11 of them (refined solve of 48 x 40 elements, n_eq 96, 12 RHS: 4.38 ms,
// now 4.03; FP64 solve of 32 x 32, n_eq 192, 1 RHS: 2.97 and 2.83 ms).
#include "internal.h"
#include "vecops.h"

namespace emsurf {
namespace {

constexpr int NT = 256;
constexpr int EPT = 4;                  // values per thread of a chunk (unless stated)
constexpr int CHUNK = NT * EPT;
constexpr int SUMS = 16;                // reals of a workgroup's combined sums

template <int CAP> struct VecList {
  VecItem it[CAP];
};

__device__ __forceinline__ double2 wave_sum(double2 v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  return v;
}

// Sums of GV complex values over the workgroup, written to out[l ostride] for
// l < count.  Each exchange step halves the values a lane holds, so 8 values
// take 17 exchanges instead of 96.
template <int GV>
__device__ __forceinline__ void block_sums(double2 (&acc)[GV], int count, double (*sh)[SUMS], double2* out,
                                           long long ostride) {
  double v[2 * GV];
#pragma unroll
  for (int i = 0; i < GV; ++i) { v[2 * i] = acc[i].x; v[2 * i + 1] = acc[i].y; }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  // after the halving, lane L holds value L / (64 / (2 GV))
#pragma unroll
  for (int half = GV, bit = 32; half >= 1; half >>= 1, bit >>= 1) {
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double keep = up ? v[i + half] : v[i], give = up ? v[i] : v[i + half];
      v[i] = keep + __shfl_xor(give, bit, 64);
    }
  }
  constexpr int LPV = 64 / (2 * GV);
#pragma unroll
  for (int bit = LPV / 2; bit >= 1; bit >>= 1) v[0] += __shfl_xor(v[0], bit, 64);
  __syncthreads();
  if (lane % LPV == 0) sh[wid][lane / LPV] = v[0];
  __syncthreads();
  if (threadIdx.x < 2 * count) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += sh[w][threadIdx.x];
    reinterpret_cast<double*>(out + (threadIdx.x >> 1) * ostride)[threadIdx.x & 1] = t;
  }
}

// one complex value per thread, summed over the workgroup into *out
__device__ __forceinline__ void block_sum(double2 v, double (*sh)[SUMS], double2* out) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) { sh[wid][0] = v.x; sh[wid][1] = v.y; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double2 r{0, 0};
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { r.x += sh[w][0]; r.y += sh[w][1]; }
    *out = r;
  }
}

// c[l] = sum of the nblk partial sums at p + l nblk, l < count: a wavefront per value
__device__ __forceinline__ void add_partials(const double2* __restrict__ p, int nblk, int count, double2* c) {
  const int lane = threadIdx.x & 63;
  for (int l = threadIdx.x >> 6; l < count; l += NT / 64) {
    double2 t{0, 0};
    for (int b = lane; b < nblk; b += 64) {
      const double2 v = p[(long long)l * nblk + b];
      t.x += v.x;
      t.y += v.y;
    }
    t = wave_sum(t);
    if (lane == 0) c[l] = t;
  }
  __syncthreads();
}

__device__ __forceinline__ void cfma_conj(double2& acc, double2 a, double2 b) {   // acc += conj(a) b
  acc.x += a.x * b.x + a.y * b.y;
  acc.y += a.x * b.y - a.y * b.x;
}
__device__ __forceinline__ void cfms(double2& acc, double2 a, double2 h) {        // acc -= a h
  acc.x -= a.x * h.x - a.y * h.y;
  acc.y -= a.x * h.y + a.y * h.x;
}

enum { DOT, UPDATE_DOT, UPDATE_NORM };

// EPT values of p from base on, this thread's share of a chunk
template <int EPT, bool FULL>
__device__ __forceinline__ void load_chunk(double2 (&w)[EPT], const double2* __restrict__ p, long long base,
                                           long long N) {
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const long long i = base + e * NT + threadIdx.x;
    w[e] = FULL || i < N ? p[i] : double2{0, 0};
  }
}
template <int EPT, bool FULL>
__device__ __forceinline__ void store_chunk(double2* p, const double2 (&w)[EPT], long long base, long long N) {
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const long long i = base + e * NT + threadIdx.x;
    if (FULL || i < N) p[i] = w[e];
  }
}

// One chunk of a step of at most GV basis vectors, all held in registers
// between the update and the dots, so that V is read once.
template <int MODE, int GV, int EPT, bool FULL>
__device__ __forceinline__ void held_chunk(const double2* __restrict__ V, long long vs, int nv, const double2* src,
                                           double2* dst, const double2* c, long long base, long long N,
                                           double2 (&acc)[GV], double2& nrm) {
  double2 w[EPT], v[GV][EPT];
  load_chunk<EPT, FULL>(w, src, base, N);
#pragma unroll
  for (int l = 0; l < GV; ++l)
    if (l < nv) load_chunk<EPT, FULL>(v[l], V + l * vs, base, N);
  if constexpr (MODE != DOT) {
#pragma unroll
    for (int l = 0; l < GV; ++l)
      if (l < nv) {
        const double2 h = c[l];
#pragma unroll
        for (int e = 0; e < EPT; ++e) cfms(w[e], v[l][e], h);
      }
    store_chunk<EPT, FULL>(dst, w, base, N);
  }
  if constexpr (MODE != UPDATE_NORM) {
#pragma unroll
    for (int l = 0; l < GV; ++l)
      if (l < nv) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) cfma_conj(acc[l], v[l][e], w[e]);
      }
  }
  if constexpr (MODE != UPDATE_DOT) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) nrm.x += w[e].x * w[e].x + w[e].y * w[e].y;
  }
}

// Partial sums of an item: [slots][nblk]; slot nv of the DOT launch and slot 0
// of the UPDATE_NORM launch hold ||.||^2.  grid (nblk, items).  HELD: nv <= GV;
// otherwise the dots read V again, GV vectors at a time.
template <int MODE, int GV, int EPT, bool HELD, int CAP>
__global__ void __launch_bounds__(NT) arnoldi_kernel(VecList<CAP> list, long long N, int nblk, int slots,
                                                     const double2* __restrict__ pin, double2* __restrict__ pout,
                                                     double2* __restrict__ rows, int rstride) {
  __shared__ double2 c[MODE == DOT ? 1 : HELD ? GV + 1 : 66];
  __shared__ double sh[NT / 64][SUMS];
  constexpr int CHUNK = NT * EPT;
  const int q = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
  const VecItem& it = list.it[q];
  const double2* V = it.V;
  const long long vs = it.vstride;
  const int nv = it.nv;
  const double2* src = MODE == UPDATE_NORM ? it.dst : it.src;
  double2* dst = it.dst;
  double2* out = pout + (long long)q * slots * nblk + blk;
  if constexpr (MODE != DOT) {
    // the coefficients (and, after the first dots, ||w||^2) of the kernel before
    const int count = nv + (MODE == UPDATE_DOT ? 1 : 0);
    add_partials(pin + (long long)q * slots * nblk, nblk, count, c);
    if (blk == 0 && tid < count) rows[(long long)it.row * rstride + tid] = c[tid];
  }
  const long long stride = (long long)nblk * CHUNK;
  double2 nrm{0, 0};
  if constexpr (HELD) {
    double2 acc[GV];
#pragma unroll
    for (int l = 0; l < GV; ++l) acc[l] = double2{0, 0};
#pragma unroll 1
    for (long long base = (long long)blk * CHUNK; base < N; base += stride) {
      if (base + CHUNK <= N)
        held_chunk<MODE, GV, EPT, true>(V, vs, nv, src, dst, c, base, N, acc, nrm);
      else
        held_chunk<MODE, GV, EPT, false>(V, vs, nv, src, dst, c, base, N, acc, nrm);
    }
    if constexpr (MODE != UPDATE_NORM) block_sums<GV>(acc, nv, sh, out, nblk);
  } else {
    if constexpr (MODE != DOT) {
      for (long long base = (long long)blk * CHUNK; base < N; base += stride) {
        double2 w[EPT], v[EPT];
        load_chunk<EPT, false>(w, src, base, N);
#pragma unroll 4
        for (int l = 0; l < nv; ++l) {
          load_chunk<EPT, false>(v, V + l * vs, base, N);
          const double2 h = c[l];
#pragma unroll
          for (int e = 0; e < EPT; ++e) cfms(w[e], v[e], h);
        }
        store_chunk<EPT, false>(dst, w, base, N);
#pragma unroll
        for (int e = 0; e < EPT; ++e) nrm.x += w[e].x * w[e].x + w[e].y * w[e].y;
      }
    }
    if constexpr (MODE != UPDATE_NORM) {
      const double2* wsrc = MODE == DOT ? src : dst;   // (this thread's own values)
      for (int g0 = 0; g0 < nv; g0 += GV) {
        double2 acc[GV], none{0, 0};
#pragma unroll
        for (int l = 0; l < GV; ++l) acc[l] = double2{0, 0};
        const int ng = nv - g0 < GV ? nv - g0 : GV;
#pragma unroll 1
        for (long long base = (long long)blk * CHUNK; base < N; base += stride)
          held_chunk<DOT, GV, EPT, false>(V + g0 * vs, vs, ng, wsrc, nullptr, nullptr, base, N, acc,
                                          MODE == DOT && g0 == 0 ? nrm : none);
        block_sums<GV>(acc, ng, sh, out + (long long)g0 * nblk, nblk);
      }
    }
  }
  if constexpr (MODE == DOT) block_sum(nrm, sh, out + (long long)nv * nblk);
  if constexpr (MODE == UPDATE_NORM) block_sum(nrm, sh, out);
}

// dst *= 1 / ||dst|| (0 at a breakdown), the norm from the partial sums p3 and
// ||w|| from slot nv of p1; rows[q rstride].x = ||dst||^2
template <int CAP>
__global__ void __launch_bounds__(NT) normalise_kernel(VecList<CAP> list, long long N, int nblk, int slots,
                                                       const double2* __restrict__ p1,
                                                       const double2* __restrict__ p3, double2* __restrict__ rows,
                                                       int rstride) {
  __shared__ double2 c[2];
  const int q = blockIdx.y, tid = threadIdx.x;
  const VecItem& it = list.it[q];
  const long long row = (long long)q * slots * nblk;
  // wavefront 0 adds up ||dst||^2, wavefront 1 ||w||^2
  if (tid < 128) {
    const double2* p = tid < 64 ? p3 + row : p1 + row + (long long)it.nv * nblk;
    double2 t{0, 0};
    for (int b = tid & 63; b < nblk; b += 64) t.x += p[b].x;
    t = wave_sum(t);
    if ((tid & 63) == 0) c[tid >> 6] = t;
  }
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0) rows[(long long)it.row * rstride] = c[0];
  const double hn = sqrt(c[0].x), wn0 = sqrt(c[1].x);
  const double f = hn <= 1e-14 * wn0 ? 0.0 : 1.0 / hn;
  for (long long i = blockIdx.x * (long long)NT + tid; i < N; i += (long long)gridDim.x * NT) {
    const double2 a = it.dst[i];
    it.dst[i] = double2{a.x * f, a.y * f};
  }
}

// partial (||w||^2, entries that are not finite) of w = src (RES: dst = w = scale (b - src))
template <bool RES, int CAP>
__global__ void __launch_bounds__(NT) norm_kernel(VecList<CAP> list, long long N, int nblk,
                                                  double2* __restrict__ pout) {
  __shared__ double sh[NT / 64][SUMS];
  const int q = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
  const VecItem& it = list.it[q];
  const bool on = it.scale != 0.0;
  double2 acc{0, 0};
  for (long long base = (long long)blk * CHUNK; base < N; base += (long long)nblk * CHUNK) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const long long i = base + e * NT + tid;
      if (i >= N) continue;
      double2 w = it.src[i];
      if constexpr (RES) {
        const double2 b = it.b[i];
        w = on ? double2{b.x - w.x, b.y - w.y} : double2{0, 0};
        it.dst[i] = w;
      } else {
        acc.y += isfinite(w.x) && isfinite(w.y) ? 0.0 : 1.0;
      }
      acc.x += w.x * w.x + w.y * w.y;
    }
  }
  block_sum(acc, sh, pout + (long long)q * nblk + blk);
}

// rows[q rstride] = sum of the nblk partial sums of item q
__global__ void __launch_bounds__(NT) add_norms_kernel(const double2* __restrict__ p, int nblk,
                                                       double2* __restrict__ rows, int rstride) {
  __shared__ double2 c[1];
  add_partials(p + (long long)blockIdx.x * nblk, nblk, 1, c);
  if (threadIdx.x == 0) rows[(long long)blockIdx.x * rstride] = c[0];
}

template <int CAP>
__global__ void __launch_bounds__(NT) scaled_copy_kernel(VecList<CAP> list, long long N) {
  const VecItem& it = list.it[blockIdx.y];
  const double f = it.scale;
  for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < N; i += (long long)gridDim.x * NT) {
    const double2 a = it.src[i];
    it.dst[i] = double2{a.x * f, a.y * f};
  }
}

template <int CAP> __global__ void __launch_bounds__(NT) solution_kernel(VecList<CAP> list, long long N) {
  const VecItem& it = list.it[blockIdx.y];
  const int nv = it.nv;
  for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < N; i += (long long)gridDim.x * NT) {
    double2 acc = it.dst[i];
#pragma unroll 4
    for (int l = 0; l < nv; ++l) {
      const double2 a = it.V[l * it.vstride + i];
      const double2 h = it.b[l];
      acc.x += a.x * h.x - a.y * h.y;
      acc.y += a.x * h.y + a.y * h.x;
    }
    it.dst[i] = acc;
  }
}

// x[i] += d[i]
__global__ void __launch_bounds__(NT) add_kernel(double2* __restrict__ x, const double2* __restrict__ d,
                                                 long long total) {
  for (long long i = blockIdx.x * (long long)NT + threadIdx.x; i < total; i += (long long)gridDim.x * NT) {
    x[i].x += d[i].x;
    x[i].y += d[i].y;
  }
}

unsigned stream_blocks(long long N) {
  long long g = (N + NT - 1) / NT;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// f(list) with the smallest argument block that holds the items
template <typename F> void with_list(const std::vector<VecItem>& items, F&& f) {
  EMS_CHECK_ARG(items.size() <= VEC_ITEMS, "internal: too many vectors in a launch");
  auto call = [&](auto list) {
    for (size_t i = 0; i < items.size(); ++i) list.it[i] = items[i];
    f(list);
  };
  if (items.size() <= 4) call(VecList<4>{});
  else if (items.size() <= 16) call(VecList<16>{});
  else call(VecList<VEC_ITEMS>{});
  EMS_LAUNCH_CHECK();
}

}  // namespace

// Chunks of 1024 values, at most 512 workgroups per vector: every workgroup of
// the next kernel adds up all partial sums, 8 KB per basis vector at 512.
int dot_blocks(long long N) {
  long long b = (N + CHUNK - 1) / CHUNK;
  if (b > 512) b = 512;
  if (b < 1) b = 1;
  return (int)b;
}

// partial sums of the first dots, the second dots and the norm
size_t vec_partial_bytes(int nq, int nv, long long N) {
  return (size_t)3 * nq * (nv + 1) * dot_blocks(N) * sizeof(double2);
}

namespace {
template <int GV, int EP, bool HELD>
void arnoldi_class(const std::vector<VecItem>& items, long long N, int slots, double2* p, double2* rows,
                   const ArnoldiRow& at, hipStream_t s) {
  if (items.empty()) return;
  const unsigned nq = (unsigned)items.size();
  const int nblk = dot_blocks(N);
  const size_t each = (size_t)nq * slots * nblk;
  double2 *p1 = p, *p2 = p + each, *p3 = p + 2 * each;
  const dim3 grid((unsigned)nblk, nq);
  with_list(items, [&](const auto& list) {
    constexpr int CAP = sizeof(list) / sizeof(VecItem);
    hipLaunchKernelGGL((arnoldi_kernel<DOT, GV, EP, HELD, CAP>), grid, dim3(NT), 0, s, list, N, nblk, slots,
                       static_cast<const double2*>(nullptr), p1, static_cast<double2*>(nullptr), 0);
    hipLaunchKernelGGL((arnoldi_kernel<UPDATE_DOT, GV, EP, HELD, CAP>), grid, dim3(NT), 0, s, list, N, nblk, slots,
                       static_cast<const double2*>(p1), p2, rows + at.o1, at.rstride);
    hipLaunchKernelGGL((arnoldi_kernel<UPDATE_NORM, GV, EP, HELD, CAP>), grid, dim3(NT), 0, s, list, N, nblk, slots,
                       static_cast<const double2*>(p2), p3, rows + at.o2, at.rstride);
    hipLaunchKernelGGL((normalise_kernel<CAP>), grid, dim3(NT), 0, s, list, N, nblk, slots,
                       static_cast<const double2*>(p1), static_cast<const double2*>(p3), rows + at.o3, at.rstride);
  });
}
}  // namespace

// The kernel of an item depends on its own basis size alone, so that its sums
// do not change with the other items: up to 2 and 4 vectors are held as 4
// values per thread, up to 8 as one (with 2 the kernels need 196 to 226
// registers and ran three times longer), more are read twice.
void launch_arnoldi(const std::vector<VecItem>& items, long long N, int nv_max, void* partial, double2* rows,
                    const ArnoldiRow& at, hipStream_t s) {
  std::vector<VecItem> cls[4];
  for (size_t q = 0; q < items.size(); ++q) {
    const int nv = items[q].nv;
    EMS_CHECK_ARG(nv >= 1 && nv <= nv_max && nv_max <= 64, "internal: basis size");
    VecItem it = items[q];
    it.row = (int)q;
    cls[nv <= 2 ? 0 : nv <= 4 ? 1 : nv <= 8 ? 2 : 3].push_back(it);
  }
  const int slots = nv_max + 1;
  const size_t per_item = (size_t)3 * slots * dot_blocks(N);
  double2* p[4] = {static_cast<double2*>(partial)};
  for (int k = 1; k < 4; ++k) p[k] = p[k - 1] + per_item * cls[k - 1].size();
  arnoldi_class<2, 4, true>(cls[0], N, slots, p[0], rows, at, s);
  arnoldi_class<4, 4, true>(cls[1], N, slots, p[1], rows, at, s);
  arnoldi_class<8, 1, true>(cls[2], N, slots, p[2], rows, at, s);
  arnoldi_class<4, 2, false>(cls[3], N, slots, p[3], rows, at, s);
}

namespace {
template <bool RES>
void norms(const std::vector<VecItem>& items, long long N, void* partial, double2* rows, int rstride, hipStream_t s) {
  if (items.empty()) return;
  const unsigned nq = (unsigned)items.size();
  const int nblk = dot_blocks(N);
  double2* p = static_cast<double2*>(partial);
  with_list(items, [&](const auto& list) {
    constexpr int CAP = sizeof(list) / sizeof(VecItem);
    hipLaunchKernelGGL((norm_kernel<RES, CAP>), dim3((unsigned)nblk, nq), dim3(NT), 0, s, list, N, nblk, p);
  });
  hipLaunchKernelGGL(add_norms_kernel, dim3(nq), dim3(NT), 0, s, static_cast<const double2*>(p), nblk, rows, rstride);
  EMS_LAUNCH_CHECK();
}
}  // namespace

void launch_norms(const std::vector<VecItem>& items, long long N, void* partial, double2* rows, int rstride,
                  hipStream_t s) {
  norms<false>(items, N, partial, rows, rstride, s);
}

void launch_residuals(const std::vector<VecItem>& items, long long N, void* partial, double2* rows, int rstride,
                      hipStream_t s) {
  norms<true>(items, N, partial, rows, rstride, s);
}

void launch_scaled_copies(const std::vector<VecItem>& items, long long N, hipStream_t s) {
  if (items.empty()) return;
  const dim3 grid(stream_blocks(N), (unsigned)items.size());
  with_list(items, [&](const auto& list) {
    constexpr int CAP = sizeof(list) / sizeof(VecItem);
    hipLaunchKernelGGL((scaled_copy_kernel<CAP>), grid, dim3(NT), 0, s, list, N);
  });
}

void launch_solutions(const std::vector<VecItem>& items, long long N, hipStream_t s) {
  if (items.empty()) return;
  const dim3 grid(stream_blocks(N), (unsigned)items.size());
  with_list(items, [&](const auto& list) {
    constexpr int CAP = sizeof(list) / sizeof(VecItem);
    hipLaunchKernelGGL((solution_kernel<CAP>), grid, dim3(NT), 0, s, list, N);
  });
}

void launch_add(void* x, const void* d, long long total, hipStream_t s) {
  hipLaunchKernelGGL(add_kernel, dim3(stream_blocks(total)), dim3(NT), 0, s, static_cast<double2*>(x),
                     static_cast<const double2*>(d), total);
  EMS_LAUNCH_CHECK();
}

}  // namespace emsurf
