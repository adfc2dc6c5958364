// Small grid kernels of the slice loop: buffer clears, the predictor-corrector
// initial guess and bookkeeping, output copies and layout conversions.
#include "common.hpp"
#include "kernels.hpp"
#include "out_body.hpp"
#include "partials.hpp"

namespace qsp {

namespace {

dim3 grid_for(size_t n) {
  size_t b = (n + kBlock - 1) / kBlock;
  if (b > 65536) b = 65536;
  if (b == 0) b = 1;
  return dim3(static_cast<unsigned>(b));
}

template <typename T>
__global__ void k_zero(T* p, size_t n) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    p[i] = T(0);
}

// explicit beam current of a slice: an ultra-relativistic beam has
// rho_b = Jz_b and rho_b - Jz_b = 0, so the plane is added to Jz (and to a
// separate rho channel if one is kept)
__global__ void k_add_current(size_t n, const double* src, double* jz, double* rho) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const double v = src[i];
    jz[i] += v;
    if (rho) rho[i] += v;
  }
}

__global__ void k_slice_end(DevCounters* ctr, int32_t* iters_out, int32_t* iters_own,
                            double* resid_out, double tol, int max_iter, int budgeted, const double* pc_partial, int pc_nblk) {
  if (pc_partial && !ctr->pc_done) partials::pc_consume(pc_partial, pc_nblk, tol, ctr, true);
  if (threadIdx.x != 0) return;
  const double r = ctr->pc_resid;
  if (iters_out) *iters_out = static_cast<int32_t>(ctr->pc_iters);
  if (iters_own) *iters_own = own_iters(ctr->pc_iters, r, tol);
  if (resid_out) *resid_out = r;
  if (r > ctr->max_resid || r != r) ctr->max_resid = r;
  if (tol > 0.0 && !ctr->pc_done) {
    if (static_cast<int>(ctr->pc_iters) >= max_iter) ctr->pc_not_converged += 1ull;
    else if (budgeted) ctr->budget_short += 1u;
  }
}

__global__ void __launch_bounds__(kBlock) k_out_copy(Geom g, OutCopy c) {
  out_detail::out_copy_all(g, c, static_cast<int>(blockIdx.x));
}

template <typename S, typename T>
__global__ void k_from_nodes(Geom g, const S* src, T* dst) {
  const size_t n = static_cast<size_t>(g.nx) * g.ny;
  for (size_t e = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; e < n;
       e += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const int i = static_cast<int>(e % g.nx), j = static_cast<int>(e / g.nx);
    const bool interior = i > 0 && j > 0;
    dst[e] = interior ? static_cast<T>(src[static_cast<size_t>(j) * (g.nx + 1) + i]) : T(0);
  }
}

template <typename T>
__global__ void k_to_nodes(Geom g, const T* src, double* dst) {
  const size_t n = static_cast<size_t>(g.nx + 1) * (g.ny + 1);
  for (size_t e = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; e < n;
       e += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const int i = static_cast<int>(e % (g.nx + 1)), j = static_cast<int>(e / (g.nx + 1));
    dst[e] = (i < g.nx && j < g.ny) ? static_cast<double>(src[static_cast<size_t>(j) * g.nx + i])
                                    : 0.0;
  }
}

}  // namespace

void launch_zero(double* p, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero<double>, grid_for(n), dim3(kBlock), 0, st, p, n);
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_zero_t(T* p, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero<T>, grid_for(n), dim3(kBlock), 0, st, p, n);
  QSP_LAUNCH_CHECK();
}

void launch_add_current(size_t n, const double* src, double* jz, double* rho, hipStream_t st) {
  hipLaunchKernelGGL(k_add_current, grid_for(n), dim3(kBlock), 0, st, n, src, jz, rho);
  QSP_LAUNCH_CHECK();
}

void launch_slice_end(DevCounters* ctr, int32_t* iters_out, int32_t* iters_own, double* resid_out,
                      double tol, int max_iter, int budgeted, const double* pc_partial, int pc_nblk,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_slice_end, dim3(1), dim3(kBlock), 0, st, ctr, iters_out, iters_own,
                     resid_out, tol, max_iter, budgeted, pc_partial, pc_nblk);
  QSP_LAUNCH_CHECK();
}

void launch_out_copy(const Geom& g, const OutCopy& c, hipStream_t st) {
  if (c.count == 0) return;
  hipLaunchKernelGGL(k_out_copy, dim3(static_cast<unsigned>(out_detail::out_wgs_all(g, c))), dim3(kBlock),
                     0, st, g, c);
  QSP_LAUNCH_CHECK();
}

template <typename S, typename T>
void launch_from_nodes(const Geom& g, const S* src, T* dst, hipStream_t st) {
  hipLaunchKernelGGL((k_from_nodes<S, T>), grid_for(static_cast<size_t>(g.nx) * g.ny), dim3(kBlock),
                     0, st, g, src, dst);
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_to_nodes(const Geom& g, const T* src, double* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_to_nodes<T>, grid_for(static_cast<size_t>(g.nx + 1) * (g.ny + 1)),
                     dim3(kBlock), 0, st, g, src, dst);
  QSP_LAUNCH_CHECK();
}

#define QSP_INST(T)                                                                       \
  template void launch_zero_t<T>(T*, size_t, hipStream_t);                                \
  template void launch_from_nodes<double, T>(const Geom&, const double*, T*, hipStream_t); \
  template void launch_to_nodes<T>(const Geom&, const T*, double*, hipStream_t);
QSP_INST(float)
QSP_INST(double)
#undef QSP_INST

}  // namespace qsp
