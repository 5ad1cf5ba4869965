// Launchers of the GMRES vector kernels (vecops.hip).  A launch works on up to
// 64 independent vectors of N c128 values, one item each; the items travel in
// the kernel arguments.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

namespace emsurf {

constexpr int VEC_ITEMS = 64;
// Meaning of an item per launch:
//   scaled copy: dst = scale src
//   residual:    dst = scale (b - src), scale 0 or 1
//   Arnoldi:     basis vectors V, V + vstride, .. (nv of them), the new vector
//                w read from src and left, orthonormalised, in dst
//   norm:        ||src||
//   solution:    dst += sum_{l < nv} V_l y_l, y = b (device)
struct VecItem {
  const double2* V = nullptr;
  const double2* src = nullptr;
  const double2* b = nullptr;
  double2* dst = nullptr;
  long long vstride = 0;
  double scale = 1.0;
  int nv = 0;
  int row = 0;   // set by the Arnoldi launch
};

// workgroups that share one vector (their partial sums are added in order)
int dot_blocks(long long N);
// bytes of the partial sums of nq items with up to nv basis vectors
size_t vec_partial_bytes(int nq, int nv, long long N);

// Row q of a result array (host memory the device writes, or device memory;
// rstride double2 values apart) after an Arnoldi step with nv basis vectors:
//   [o1 + l]  first coefficients c1 = V_l^H w, [o1 + nv].x = ||w||^2
//   [o2 + l]  second coefficients V_l^H (w - V c1)
//   [o3].x    ||w - V (c1 + c2)||^2
// dst receives the remainder divided by its norm, or zero where the norm is
// at most 1e-14 ||w|| (the solver's breakdown rule).
struct ArnoldiRow {
  int o1, o2, o3, rstride;
};
void launch_arnoldi(const std::vector<VecItem>& items, long long N, int nv_max, void* partial, double2* rows,
                    const ArnoldiRow& at, hipStream_t s);
// rows[q rstride] = (||src||^2, number of entries of src that are not finite)
void launch_norms(const std::vector<VecItem>& items, long long N, void* partial, double2* rows, int rstride,
                  hipStream_t s);
// dst = scale (b - src), rows[q rstride].x = ||dst||^2
void launch_residuals(const std::vector<VecItem>& items, long long N, void* partial, double2* rows, int rstride,
                      hipStream_t s);
void launch_scaled_copies(const std::vector<VecItem>& items, long long N, hipStream_t s);
void launch_solutions(const std::vector<VecItem>& items, long long N, hipStream_t s);
// x += d, total values
void launch_add(void* x, const void* d, long long total, hipStream_t s);

}  // namespace emsurf
