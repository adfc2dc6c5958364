// Shared declarations of the libqsp runtime and its HIP kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <stdexcept>
#include <string>

namespace qsp {

// 256 threads = 4 wave64 wavefronts per workgroup everywhere.
constexpr int kBlock = 256;

// Largest number of output copies one slice can request (12 quantities as
// full plane, centre row and axis node).
constexpr int kMaxOut = 36;

// Fifth-order Adams-Bashforth weights (numerators over 720) for
// f_k, f_{k-1}, ..., f_{k-4}.
constexpr double kAB5[5] = {1901.0 / 720.0, -2774.0 / 720.0, 2616.0 / 720.0,
                            -1274.0 / 720.0, 251.0 / 720.0};

// History part of an Adams-Bashforth step from slice k: y_k - dz (b1 f_{k-1}
// + b2 f_{k-2} + b3 f_{k-3} + b4 f_{k-4}), so that y_{k+1} = P_k - dz b0 f_k.
// One function for every place that forms it (the real push, state import,
// checkpoint restore), so that they round alike.
template <typename T>
__host__ __device__ __forceinline__ T ab5_history(T y, T f1, T f2, T f3, T f4, T dz) {
  return y - dz * (T(kAB5[1]) * f1 + T(kAB5[2]) * f2 + T(kAB5[3]) * f3 + T(kAB5[4]) * f4);
}

struct DeviceError : std::runtime_error {
  using std::runtime_error::runtime_error;
};

inline void hip_check(hipError_t e, const char* what, const char* file, int line) {
  if (e != hipSuccess) {
    char buf[512];
    std::snprintf(buf, sizeof(buf), "%s failed at %s:%d: %s", what, file, line,
                  hipGetErrorString(e));
    throw DeviceError(buf);
  }
}
#define QSP_HIP(call) ::qsp::hip_check((call), #call, __FILE__, __LINE__)
#define QSP_LAUNCH_CHECK() ::qsp::hip_check(hipGetLastError(), "kernel launch", __FILE__, __LINE__)

template <typename T>
struct Cplx {
  T re, im;
};

// ---------------------------------------------------------------------------
// Grid geometry shared by all kernels.  Node arrays are stored [ny][nx]
// (pitch nx): element (j, i) is node (i, j) for i, j in 0..n-1; node index 0
// carries the Dirichlet boundary (always 0 for fields) and node index n is
// implicit (0).  This makes each stored row the first half of the odd
// extension a type-I sine transform needs.
// ---------------------------------------------------------------------------
struct Geom {
  int nx, ny;            // cells = nodes per stored row/column
  int lx, ly;            // log2(nx), log2(ny)
  double x_lo, y_lo, hx, hy;
  int rr;                // rows per workgroup of the transform row passes
  int order;             // transverse particle shape order, 0..3
  // 1: the planes between the row and column passes of a solve are stored
  // in strips of 4 columns, element (j, i) at ((i / 4) ny + j) 4 + i % 4
  // (FP32 at 1024^2: the column pass reads and writes one contiguous
  // block per strip, the row passes 64-byte blocks of 4 rows x 4 columns);
  // 0: row-major
  int strip;
};

// base[i] with the byte offset formed in 32 bits (the caller guarantees
// i * sizeof(T) < 2^32), so that a uniform base loads or stores through one
// VGPR of offset instead of a 64-bit address per lane
template <typename T>
__device__ __forceinline__ T load_at(const T* base, unsigned int i) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                     i * static_cast<unsigned int>(sizeof(T)));
}
template <typename T>
__device__ __forceinline__ void store_at(T* base, unsigned int i, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + i * static_cast<unsigned int>(sizeof(T))) = v;
}

// Plasma lattice: (nx*ppc_x) x (ny*ppc_y) sites, particle p = I + J*nX.
struct Lattice {
  int nX, nY, ppc_x, ppc_y;
  int64_t np;
};

// Which transform rows of n points use, by element size (see dst_impl.hpp):
//   symmetric core   FP64 from 128, FP32 from 1024 points up: the FFT of the
//                    odd extension with its redundant half left out;
//   wave core        FP32 of 256 and 512 points: the whole odd extension,
//                    one wave per row pair.  These sizes are bound by the
//                    length of a lane's chain, which the symmetric core does
//                    not shorten;
//   matrix core      16-64 points, FP32 also 128: a product with the sine
//                    matrix.  At 128 points (128^2 box) it takes 6.8 ms
//                    in FP32, 6.0 with the symmetric core, whose Ex - By errs
//                    up to 1.25 times as much as the half-length FFT's (8.0
//                    ms) did; in FP64 7.1 against 6.8.
__host__ __device__ constexpr bool sym_core(int elem_size, int n) {
  return n >= 1024 || (elem_size == 8 && n >= 128);
}
__host__ __device__ constexpr bool wave_core(int elem_size, int n) {
  return elem_size == 4 && (n == 256 || n == 512);
}

// Rows (columns) a workgroup of the symmetric core transforms in the row
// (column) passes.
__host__ __device__ constexpr int sym_rows(int n) { return n >= 2048 ? 2 : 4; }
__host__ __device__ constexpr int sym_cols(int n) { return n >= 2048 ? 2 : 4; }

// Shape of the matrix core's products (see Dense in dst_impl.hpp): rows folded
// onto n / 2 operands (from 32 points up), operands per lane, and the output
// that column c of tile t holds.
__host__ __device__ constexpr bool dense_fold(int n) { return n >= 32; }
__host__ __device__ constexpr int dense_lane(int n) { return (dense_fold(n) ? n / 2 : n) / 4; }
__host__ __device__ constexpr int dense_out(int n, int t, int c) {
  return dense_fold(n) ? 2 * (16 * (t >> 1) + c) + (t & 1) : c;
}

// Per-axis transform tables (device pointers): for the matrix core tw holds
// 2n doubles sin(pi a / n) (exactly 0 for multiples of n; see dense_angle) and
// pre is unused; for the wave core tw[k1 * 64 + l] = e^{-2 pi i l k1 / 2n} (2n entries) and pre holds
// the complex table W_64^{la c1} at [la * 9 + c1] (la < 8, c1 < 8, entry 8 of
// a row 0); for the symmetric core tw as in sym_table_* and pre unused.
template <typename T>
struct AxisTables {
  const Cplx<T>* tw;
  const T* pre;
  const double* lam;     // Laplacian eigenvalue of sine mode p, p = 0..n-1 (0 unused)
};

// Table of the symmetric core in AxisTables::tw, H = n / 16, G = max(1, H / 8):
// entries m < 9 H: W_2n^{l k} at m = k H + l; then 16 G entries W_2H^{g c} at
// m = 9 H + 16 g + c; then 9 x 8 values sin(pi (2 j + 1) k / 16) as the real
// parts at m = 9 H + 16 G + 8 k + j.  sym_table_angle gives entry m's angle
// in units of pi (e^{-i pi angle}, or sin(pi angle) for the last part).
__host__ __device__ constexpr int sym_g(int n) { return n / 16 >= 8 ? n / 128 : 1; }
__host__ __device__ constexpr int sym_table_w(int n) { return 9 * (n / 16); }
__host__ __device__ constexpr int sym_table_s(int n) { return sym_table_w(n) + 16 * sym_g(n); }
__host__ __device__ constexpr int sym_table_size(int n) { return sym_table_s(n) + 72; }
__host__ __device__ inline double sym_table_angle(int n, int m) {
  const int H = n / 16;
  if (m < sym_table_w(n)) return static_cast<double>((m % H) * (m / H)) / n;
  if (m < sym_table_s(n)) {
    const int q = m - sym_table_w(n);
    return static_cast<double>((q / 16) * (q % 16)) / H;
  }
  const int q = m - sym_table_s(n);
  return static_cast<double>(((2 * (q % 8) + 1) * (q / 8)) % 32) / 16.0;
}

// Matrix core: entry of its table (sines of pi a / n for a = 0 .. 2n - 1, in
// FP64 for both precisions) that is lane l's operand s for tile t: output o
// times the operand index, which for the folded pair 0 means row entry n / 2
// (nothing for the even outputs: the sine of a multiple of pi).
__host__ __device__ constexpr int dense_angle(int n, int t, int l, int s) {
  const int o = dense_out(n, t, l % 16), k = dense_lane(n) * (l / 16) + s;
  return (o * (dense_fold(n) && k == 0 ? n / 2 : k)) & (2 * n - 1);
}

// Grids whose solves run in one workgroup per field (small.hip): batches on
// node arrays up to 64 x 64 (one launch of 9.7 us against three that take 11.7
// eagerly, FP32; 11.3 in FP64), the slice loop's up to 2048 nodes (32 x 64 box:
// 3.52 ms against 4.01; at 64 x 64 one CU's loads and products take longer than
// three passes' launches from a graph, 4.36 against 4.30 ms with all sums in
// FP32, 5.6 against 4.7 in FP64).
__host__ __device__ constexpr bool small_solve(int nx, int ny) { return nx <= 64 && ny <= 64; }
__host__ __device__ constexpr bool small_grid(int nx, int ny) {
  return small_solve(nx, ny) && nx * ny <= 2048;
}

// Device-side scalars of the predictor-corrector and counters.
struct DevCounters {
  unsigned int pc_done;        // 1 once the current slice's P-C converged
  unsigned int pc_iters;       // iterations done for the current slice
  unsigned int nonfinite;      // sticky: non-finite residual or norm seen
  double pc_resid;             // last residual of the current slice
  double max_resid;            // largest final residual over slices
  unsigned long long n_clamped;
  unsigned long long n_absorbed;
  unsigned long long n_dep_global;
  unsigned long long pc_iterations;
  unsigned long long pc_not_converged;
  // slices whose launched iterations (a launch budget below the maximum)
  // ended before the predictor-corrector converged
  unsigned int budget_short;
  unsigned int reserved0;
};

// What the library keeps of a slice's iterations: their count (at most 1000),
// and whether the last residual lies within a factor of ten of the tolerance.
constexpr int32_t kNearTol = 1 << 16;
__device__ inline int32_t own_iters(unsigned int iters, double resid, double tol) {
  return static_cast<int32_t>(iters) | (resid > 0.1 * tol ? kNearTol : 0);
}

}  // namespace qsp
