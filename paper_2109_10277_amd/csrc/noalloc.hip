// Batched 2D Dirichlet solve that allocates no device memory: the
// transforms' intermediate planes and their tables live in one file-scope
// static device array per GPU instead of a context's buffers (for callers
// that cannot allocate: code under stream capture, tight serving loops).
// Same three sine-transform passes as qsp_solve_poisson (fast Poisson
// solver of HiPACE++, arXiv:2109.10277 Sec. III.B), run in place.
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "kernels.hpp"
#include "runtime.hpp"

namespace {

// Planes of the solve (nbatch x nx x ny values of the field precision), then
// the two axes' tables.
constexpr size_t kPlaneBytes = size_t(16) << 20;
constexpr size_t kTableBytes = size_t(256) << 10;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kPlaneBytes + kTableBytes];

std::mutex g_mu;
unsigned char* g_ptr[kMaxDevices] = {};   // device address of `scratch`, per GPU

// Address of this device's copy of `scratch` (the device must be current).
unsigned char* scratch_on(int device) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      throw qsp::DeviceError(std::string("hipGetSymbolAddress(scratch) failed: ") +
                             hipGetErrorString(e));
    g_ptr[device] = static_cast<unsigned char*>(p);
  }
  return g_ptr[device];
}

// The transform tables of the two axes (layout as the context's, see
// AxisTables), computed on the device, one thread per entry and one grid row
// per axis.
template <typename T>
struct AxisJob {
  int n;
  double h;
  qsp::Cplx<T>* tw;
  T* pre;
  double* lam;
};

template <typename T>
__global__ void k_axis_tables(AxisJob<T> x, AxisJob<T> y) {
  const AxisJob<T> q = blockIdx.y == 0 ? x : y;
  const int n = q.n;
  qsp::Cplx<T>* tw = q.tw;
  T* pre = q.pre;
  double* lam = q.lam;
  const double h = q.h;
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  double s, c;
  if (qsp::sym_core(sizeof(T), n)) {
    if (m < qsp::sym_table_size(n)) {
      sincospi(qsp::sym_table_angle(n, m), &s, &c);
      tw[m] = m < qsp::sym_table_s(n) ? qsp::Cplx<T>{static_cast<T>(c), static_cast<T>(-s)}
                                      : qsp::Cplx<T>{static_cast<T>(s), T(0)};
    }
  } else if (qsp::wave_core(sizeof(T), n)) {
    const int k1 = m / 64, l = m % 64;
    if (m >= 2 * n) return;
    sincospi(-2.0 * static_cast<double>((l * k1) % (2 * n)) / (2 * n), &s, &c);
    tw[m] = {static_cast<T>(c), static_cast<T>(s)};
    if (m < 72) {
      auto* w = reinterpret_cast<qsp::Cplx<T>*>(pre);
      const int la = m / 9, c1 = m % 9;
      sincospi(-2.0 * (la * c1) / 64.0, &s, &c);
      w[m] = c1 < 8 ? qsp::Cplx<T>{static_cast<T>(c), static_cast<T>(s)}
                    : qsp::Cplx<T>{T(0), T(0)};
    }
  } else if (m < 2 * n) {
    reinterpret_cast<double*>(tw)[m] = m % n ? sinpi(static_cast<double>(m) / n) : 0.0;
  }
  if (m < n) {
    const double sm = sinpi(0.5 * m / n);
    lam[m] = -4.0 / (h * h) * sm * sm;
  }
}

template <typename T>
size_t axis_table_bytes(int n) {
  return static_cast<size_t>(2 * n) * sizeof(qsp::Cplx<T>) +
         static_cast<size_t>(n) * (sizeof(T) + sizeof(double));
}

template <typename T>
qsp::AxisTables<T> axis_at(unsigned char* base, int n) {
  auto* tw = reinterpret_cast<qsp::Cplx<T>*>(base);
  auto* pre = reinterpret_cast<T*>(tw + 2 * n);
  auto* lam = reinterpret_cast<double*>(pre + n);
  return {tw, pre, lam};
}

template <typename T>
void solve(const qsp_config& c, unsigned char* ptr, int nb, const T* src, T* dst, double shift,
           hipStream_t st) {
  using namespace qsp;
  Geom g{};
  g.nx = c.nx;
  g.ny = c.ny;
  for (g.lx = 0; (1 << g.lx) < c.nx; ++g.lx) {}
  for (g.ly = 0; (1 << g.ly) < c.ny; ++g.ly) {}
  g.x_lo = c.x_lo;
  g.y_lo = c.y_lo;
  g.hx = (c.x_hi - c.x_lo) / c.nx;
  g.hy = (c.y_hi - c.y_lo) / c.ny;
  g.rr = row_rows<T>(c.nx);
  g.order = 1;
  g.strip = 0;   // the passes run in place: the planes stay row-major
  T* planes = reinterpret_cast<T*>(ptr);
  unsigned char* tab = ptr + kPlaneBytes;
  // tables are 8-byte aligned pieces: x axis first, then y
  const AxisTables<T> tx = axis_at<T>(tab, c.nx);
  const AxisTables<T> ty = axis_at<T>(tab + axis_table_bytes<T>(c.nx), c.ny);
  const AxisJob<T> jx{c.nx, g.hx, const_cast<Cplx<T>*>(tx.tw), const_cast<T*>(tx.pre),
                      const_cast<double*>(tx.lam)};
  const AxisJob<T> jy{c.ny, g.hy, const_cast<Cplx<T>*>(ty.tw), const_cast<T*>(ty.pre),
                      const_cast<double*>(ty.lam)};
  const int nmax = c.nx > c.ny ? c.nx : c.ny;
  hipLaunchKernelGGL(k_axis_tables<T>, dim3((2 * nmax + 255) / 256, 2), dim3(256), 0, st, jx, jy);
  QSP_LAUNCH_CHECK();
  if (small_batch(g, src, dst, nb)) {
    launch_small_nodes<T>(g, src, dst, nb, shift, tx, ty, st);
    return;
  }
  // each pass reads its rows or column strips into LDS before writing them
  // back, so all three work on the same planes
  NodeRowArgs<T> r{src, dst, planes};
  launch_row_nodes<T>(g, r, false, nb, tx, st);
  ColArgs<T> col{};
  col.in = planes;
  col.out = planes;
  for (int b = 0; b < 4; ++b) col.shift[b] = shift;
  col.w = col_width<T>(g);
  launch_col_solve<T>(g, col, nb, ty, tx.lam, nullptr, st);
  launch_row_nodes<T>(g, r, true, nb, tx, st);
}

bool pow2_in(int v, int lo, int hi) { return v >= lo && v <= hi && (v & (v - 1)) == 0; }

}  // namespace

namespace qsp {

qsp_status solve_poisson_noalloc(const qsp_config* cfg, int device, void* stream, int nbatch,
                                 const void* src, void* dst, double shift, std::string& err) {
  if (!cfg) return err = "null config", QSP_ERR_INVALID_ARG;
  const qsp_config& c = *cfg;
  if (!pow2_in(c.nx, 16, 2048) || !pow2_in(c.ny, 16, 2048))
    return err = "nx and ny must be powers of two in [16, 2048]", QSP_ERR_INVALID_ARG;
  if (!(std::isfinite(c.x_lo) && std::isfinite(c.x_hi) && c.x_hi > c.x_lo &&
        std::isfinite(c.y_lo) && std::isfinite(c.y_hi) && c.y_hi > c.y_lo))
    return err = "box extents must be finite with hi > lo", QSP_ERR_INVALID_ARG;
  if (c.precision != QSP_FP32 && c.precision != QSP_FP64)
    return err = "precision must be QSP_FP32 or QSP_FP64", QSP_ERR_INVALID_ARG;
  if (nbatch < 1 || nbatch > 4) return err = "nbatch must be 1..4", QSP_ERR_INVALID_ARG;
  if (!(shift >= 0.0) || !std::isfinite(shift))
    return err = "shift must be finite and >= 0", QSP_ERR_INVALID_ARG;
  if (!src || !dst) return err = "null src or dst", QSP_ERR_INVALID_ARG;
  const size_t es = c.precision == QSP_FP64 ? sizeof(double) : sizeof(float);
  const size_t need = static_cast<size_t>(nbatch) * c.nx * c.ny * es;
  if (need > kPlaneBytes)
    return err = "nbatch * nx * ny values (" + std::to_string(need) +
                 " bytes) exceed the static scratch of " + std::to_string(kPlaneBytes) +
                 " bytes",
           QSP_ERR_INVALID_ARG;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev ||
      device >= kMaxDevices)
    return err = "no such HIP device", QSP_ERR_INVALID_ARG;
  try {
    QSP_HIP(hipSetDevice(device));
    unsigned char* ptr = scratch_on(device);
    const hipStream_t st = static_cast<hipStream_t>(stream);
    if (c.precision == QSP_FP64)
      solve<double>(c, ptr, nbatch, static_cast<const double*>(src), static_cast<double*>(dst),
                    shift, st);
    else
      solve<float>(c, ptr, nbatch, static_cast<const float*>(src), static_cast<float*>(dst),
                   shift, st);
  } catch (const std::exception& e) {
    err = e.what();
    return QSP_ERR_DEVICE;
  }
  return QSP_OK;
}

}  // namespace qsp
