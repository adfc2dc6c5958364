// Whole 2D solves in one workgroup per field, for the smallest grids (gfx950;
// the sizes: small_solve, small_grid).  The three passes of such a solve
// (dst_impl.hpp) are bound by their launches and by one memory round trip each,
// not by work: at 32^2 to 64^2 in FP32 they take 3.6 + 3.7 + 3.6 us for at most
// 2 MFLOP.  Here the field stays in LDS from its source to its epilogue: four
// products with the folded sine matrices (Dense), one 16x16 output tile per
// wave and product.  Measured (FP32): 32^2 box of 64 slices 3.77 -> 2.72 ms, its
// gradient run 17.0 -> 13.6, one solve at 64^2 11.7 -> 9.7 us, at 32^2 11.6 ->
// 4.4.
#include <stdexcept>

#include "common.hpp"
#include "dst_impl.hpp"
#include "kernels.hpp"

namespace qsp {
namespace {

using namespace dst_detail;

template <typename T, int LX, int LY>
struct Small {
  using X = Dense<T, LX>;
  using Y = Dense<T, LY>;
  static constexpr int nx = 1 << LX, ny = 1 << LY;
  static constexpr int NTX = X::NT, NTY = Y::NT;
  static constexpr int BS = 64 * NTX * NTY;       // threads: a wave per tile
  static constexpr int N = nx * ny / BS;          // elements per thread (4)
  static constexpr int PX = X::pitch, PY = Y::pitch;
  // T units of one of the two LDS buffers, which hold the field by rows j
  // (pitch PX) or by columns (pitch PY)
  static constexpr int size = ny * PX > nx * PY ? ny * PX : nx * PY;
  static constexpr size_t lds = 2 * size * sizeof(T);   // above 64 KiB only at 64 x 64 in FP64

  // the lane's operands of both axes and its eigenvalues, fetched behind the
  // source
  struct Op {
    double x[X::KL], y[Y::KL];
    double lx[4], ly;
  };
  static __device__ __forceinline__ Op load(const AxisTables<T>& tx, const AxisTables<T>& ty) {
    Op q;
    const int wave = static_cast<int>(threadIdx.x) >> 6, lane = static_cast<int>(threadIdx.x) & 63;
    X::load_tile(tx.tw, wave % NTX, q.x);
    Y::load_tile(ty.tw, wave % NTY, q.y);
#pragma unroll
    for (int r = 0; r < 4; ++r) q.lx[r] = tx.lam[16 * (wave / NTY) + X::template row_of<true>(lane, r)];
    q.ly = ty.lam[dense_out(ny, wave % NTY, lane & 15)];
    return q;
  }

  // position of node (i, j) in the buffer by rows
  static __device__ __forceinline__ int at(int i, int j) { return j * PX + X::ridx(i); }

  // (Dxx + Dyy - shift) u = f: f by rows in `a`, whose row 0 and column 0 are
  // zero, is replaced by u; `b` is scratch.  Row 0 and column 0 of u are products
  // with zeros, not zero for an infinity or a NaN in f: they are stored as zero
  // (selects here, inside the chain, take a solve at 64^2 from 9.66 to 9.85 us).
  // Starts and ends with a barrier.
  static __device__ __forceinline__ void solve(T* a, T* b, const Op& q, double shift) {
    const int wave = static_cast<int>(threadIdx.x) >> 6, lane = static_cast<int>(threadIdx.x) & 63;
    const int rx = wave / NTX, ox = wave % NTX;   // rows j, outputs along x
    const int ry = wave / NTY, oy = wave % NTY;   // columns, outputs along y
    const int kx = dense_out(nx, ox, lane & 15), ky = dense_out(ny, oy, lane & 15);
    // 1 / normalisation (nx ny / 4, exact): the eigenvalue sum in FP64, the one
    // division in the field precision
    const double inorm = 0.25 * nx * ny;
    T den[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) den[r] = static_cast<T>((q.lx[r] + (q.ly - shift)) * inorm);
    __syncthreads();
    const auto f1 = X::template product<true>(a + 16 * rx * PX, q.x, ox & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) b[kx * PY + Y::ridx(16 * rx + X::template row_of<true>(lane, r))] = static_cast<T>(f1[r]);
    __syncthreads();
    const auto f2 = Y::template product<true>(b + 16 * ry * PY, q.y, oy & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = 16 * ry + X::template row_of<true>(lane, r);
      const T z = static_cast<T>(f2[r]) / den[r];
      a[col * PY + Y::ridx(ky)] = col > 0 && ky > 0 ? z : T(0);
    }
    __syncthreads();
    const auto f3 = Y::template product<false>(a + 16 * ry * PY, q.y, oy & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) b[ky * PX + X::ridx(16 * ry + X::template row_of<false>(lane, r))] = static_cast<T>(f3[r]);
    __syncthreads();
    const auto f4 = X::template product<false>(b + 16 * rx * PX, q.x, ox & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) a[at(kx, 16 * rx + X::template row_of<false>(lane, r))] = static_cast<T>(f4[r]);
    __syncthreads();
  }
};

// One corrector solve of Bx (FX) or By: source, solve, update of the iterate
// with its residual sums, and the clearing of the trial plane of the field's
// own channel, which the source has just read.
template <typename T, int LX, int LY, bool FX>
__device__ __forceinline__ void small_bxby(const Geom& g, const SrcBxBy<T>& s, const PCArgs<T>& pc,
                                           const ZeroJob& z, const AxisTables<T>& tx,
                                           const AxisTables<T>& ty, T* a) {
  using S = Small<T, LX, LY>;
  constexpr int nx = S::nx, ny = S::ny, N = S::N;
  T* b = a + S::size;
  const int t = static_cast<int>(threadIdx.x);
  const double* __restrict__ prev = FX ? s.jy_prev : s.jx_prev;
  const double* __restrict__ next = FX ? s.jy_next : s.jx_next;
  const double* __restrict__ shrd = FX ? s.sy_next : s.sx_next;
  T* field = FX ? pc.bx : pc.by;
  T* tape = FX ? pc.tape_bx : pc.tape_by;
  // source: -d_y Jz + d_zeta Jy - shift Bx_old for Bx, d_x Jz - d_zeta Jx -
  // shift By_old for By, neighbours with clamped indices; the Gaussian beam's
  // Jz from its profile factors across (gc) and along (g0, g1) the derivative
  double z0[N], z1[N], p[N], q[N], h[N], gc[N], g0[N], g1[N];
  T old_b[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    z0[u] = load_at(s.jz, FX ? (j > 0 ? e - nx : e) : (i > 0 ? e - 1 : e));
    z1[u] = load_at(s.jz, FX ? (j + 1 < ny ? e + nx : e) : (i + 1 < nx ? e + 1 : e));
    p[u] = load_at(prev, e);
    q[u] = load_at(next, e);
    h[u] = load_at(shrd, e);
    old_b[u] = load_at(static_cast<const T*>(field), e);
    gc[u] = FX ? load_at(s.bgx, i) : load_at(s.bgy, j);
    g0[u] = FX ? load_at(s.bgy, j > 0 ? j - 1 : 0) : load_at(s.bgx, i > 0 ? i - 1 : 0);
    g1[u] = FX ? load_at(s.bgy, j + 1) : load_at(s.bgx, i + 1);
  }
  __builtin_amdgcn_sched_barrier(0);
  auto op = S::load(tx, ty);   // behind the source: needed last
  __builtin_amdgcn_sched_barrier(0);
  const double ih = FX ? -0.5 / g.hy : 0.5 / g.hx;
  const double idz = FX ? 0.5 / s.dzeta : -0.5 / s.dzeta;
  const double amp = s.beam_amp;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    pin(z0[u]);
    pin(z1[u]);
    pin(p[u]);
    pin(q[u]);
    pin(h[u]);
    pin(old_b[u]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    const double q0 = z0[u] - amp * gc[u] * g0[u];
    const double q1 = (FX ? j + 1 < ny : i + 1 < nx) ? z1[u] - amp * gc[u] * g1[u] : 0.0;
    const double v =
        (q1 - q0) * ih + (p[u] - (q[u] + h[u])) * idz - s.shift * static_cast<double>(old_b[u]);
    a[S::at(i, j)] = static_cast<T>((i > 0 && j > 0) ? v : 0.0);
  }
  double* clear = z.p[FX ? 1 : 0];   // each thread clears what it has read
#pragma unroll
  for (int u = 0; u < N; ++u) store_at(clear, t + u * S::BS, 0.0);
  S::solve(a, b, op, s.shift);
  double dsum = 0.0, nsum = 0.0;
  T v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    v[u] = i > 0 && j > 0 ? a[S::at(i, j)] : T(0);
    const double d = static_cast<double>(v[u]) - static_cast<double>(old_b[u]);
    dsum += d * d;
    nsum += static_cast<double>(v[u]) * static_cast<double>(v[u]);
    store_at(field, e, v[u]);
  }
  if (tape)
#pragma unroll
    for (int u = 0; u < N; ++u) store_at(tape, t + u * S::BS, v[u]);
  __shared__ double red[2][16];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    dsum += __shfl_down(dsum, off, 64);
    nsum += __shfl_down(nsum, off, 64);
  }
  if ((t & 63) == 0) {
    red[0][t >> 6] = dsum;
    red[1][t >> 6] = nsum;
  }
  __syncthreads();
  if (t < 2) {
    double sum = 0.0;
    for (int w = 0; w < S::BS / 64; ++w) sum += red[t][w];
    pc.partial[(FX ? 0 : 2) + t] = sum;
  }
}

template <typename T, int LX, int LY>
__global__ void __launch_bounds__((Small<T, LX, LY>::BS))
k_small_bxby(Geom g, SrcBxBy<T> s, PCArgs<T> pc, ZeroJob z, AxisTables<T> tx, AxisTables<T> ty,
             const DevCounters* ctr) {
  if (ctr->pc_done) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* a = reinterpret_cast<T*>(smem_raw);
  if (blockIdx.x == 0)
    small_bxby<T, LX, LY, true>(g, s, pc, z, tx, ty, a);
  else
    small_bxby<T, LX, LY, false>(g, s, pc, z, tx, ty, a);
}

// psi (blockIdx.x = 0, with Ex - By and Ey + Bx from its differences), Ez (1)
// and Bz (2) of a slice; the initial guess of the predictor-corrector (3);
// then one workgroup per plane to clear.
template <typename T, int LX, int LY>
__global__ void __launch_bounds__((Small<T, LX, LY>::BS))
k_small_pez(Geom g, SrcPEZ<T> s, RowInvArgs<T> r, ZeroJob z, AxisTables<T> tx, AxisTables<T> ty) {
  using S = Small<T, LX, LY>;
  constexpr int nx = S::nx, ny = S::ny, N = S::N;
  const int fld = blockIdx.x;
  const int t = static_cast<int>(threadIdx.x);
  if (fld > 3) {
#pragma unroll
    for (int c = 0; c < 8; ++c)   // plane pointers by constant index: kernel arguments
      if (c == fld - 4)
#pragma unroll
        for (int u = 0; u < N; ++u) store_at(z.p[c], t + u * S::BS, 0.0);
    return;
  }
  if (fld == 3) {
    static_assert(N <= kGuess, "one batch of the guess covers the plane");
    GuessRegs<T> gr;
    guess_load(r.guess, size_t(nx) * ny, size_t(t), size_t(S::BS), gr);
    guess_store(r.guess, size_t(nx) * ny, size_t(t), size_t(S::BS), gr);
    if (t == 0) {
      r.guess.ctr->pc_done = 0u;
      r.guess.ctr->pc_iters = 0u;
      r.guess.ctr->pc_resid = 0.0;
    }
    return;
  }
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* a = reinterpret_cast<T*>(smem_raw);
  T* b = a + S::size;
  typename S::Op op;
  // psi: -(rho - Jz + ions); Ez: d_x Jx + d_y Jy; Bz: d_y Jx - d_x Jy
  if (fld == 0) {
    double v[N], w[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int e = t + u * S::BS;
      v[u] = load_at(s.rho_mjz, e);
      w[u] = s.n0;
    }
    op = S::load(tx, ty);
    if (s.ionx) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int e = t + u * S::BS;
        w[u] *= load_at(s.ionx, e & (nx - 1)) * load_at(s.iony, e >> LX);
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
      a[S::at(i, j)] = static_cast<T>((i > 0 && j > 0) ? -(v[u] + w[u]) : 0.0);
    }
  } else {
    const double ihx = fld == 1 ? 0.5 / g.hx : -0.5 / g.hx, ihy = 0.5 / g.hy;
    const double* __restrict__ ax = fld == 1 ? s.jx : s.jy;
    const double* __restrict__ ay = fld == 1 ? s.jy : s.jx;
    double ve[N], vw[N], vn[N], vs[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
      ve[u] = load_at(ax, i + 1 < nx ? e + 1 : e);
      vw[u] = load_at(ax, i > 0 ? e - 1 : e);
      vn[u] = load_at(ay, j + 1 < ny ? e + nx : e);
      vs[u] = load_at(ay, j > 0 ? e - nx : e);
    }
    __builtin_amdgcn_sched_barrier(0);
    op = S::load(tx, ty);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      pin(ve[u]);
      pin(vw[u]);
      pin(vn[u]);
      pin(vs[u]);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
      const double v = ((i + 1 < nx ? ve[u] : 0.0) - vw[u]) * ihx + ((j + 1 < ny ? vn[u] : 0.0) - vs[u]) * ihy;
      a[S::at(i, j)] = static_cast<T>((i > 0 && j > 0) ? v : 0.0);
    }
  }
  S::solve(a, b, op, 0.0);
  T* out = fld == 0 ? r.out[0] : (fld == 1 ? r.out[2] : r.out[3]);
  const T mihx = static_cast<T>(-0.5 / g.hx), mihy = static_cast<T>(-0.5 / g.hy);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    const bool in = i > 0 && j > 0;
    store_at(out, e, in ? a[S::at(i, j)] : T(0));
    if (fld == 0) {
      // central differences, zero on row and column 0 and beyond the grid
      const T ue = i + 1 < nx ? a[S::at(i + 1 < nx ? i + 1 : i, j)] : T(0), uw = a[S::at(i > 0 ? i - 1 : 0, j)];
      const T un = j + 1 < ny ? a[S::at(i, j + 1 < ny ? j + 1 : j)] : T(0), us = a[S::at(i, j > 0 ? j - 1 : 0)];
      store_at(r.out_dx[0], e, in ? mihx * (ue - uw) : T(0));
      store_at(r.out[1], e, in ? mihy * (un - us) : T(0));
    }
  }
}

// A batch of solves on node arrays, one workgroup per solve (a workgroup reads
// its sources before it writes; see small_batch for several).
template <typename T, int LX, int LY>
__global__ void __launch_bounds__((Small<T, LX, LY>::BS))
k_small_nodes(const T* src, T* dst, double shift, AxisTables<T> tx, AxisTables<T> ty) {
  using S = Small<T, LX, LY>;
  constexpr int nx = S::nx, ny = S::ny, N = S::N;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* a = reinterpret_cast<T*>(smem_raw);
  T* b = a + S::size;
  const int t = static_cast<int>(threadIdx.x);
  const size_t nodes = static_cast<size_t>(nx + 1) * (ny + 1);
  src += blockIdx.x * nodes;
  dst += blockIdx.x * nodes;
  T v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS;
    v[u] = load_at(src, (e >> LX) * (nx + 1) + (e & (nx - 1)));
  }
  const auto op = S::load(tx, ty);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    a[S::at(i, j)] = i > 0 && j > 0 ? v[u] : T(0);   // boundary nodes count as zero
  }
  S::solve(a, b, op, shift);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = t + u * S::BS, i = e & (nx - 1), j = e >> LX;
    store_at(dst, j * (nx + 1) + i, i > 0 && j > 0 ? a[S::at(i, j)] : T(0));
  }
  if (t < ny) dst[t * (nx + 1) + nx] = T(0);
  for (int i = t; i <= nx; i += S::BS) dst[ny * (nx + 1) + i] = T(0);
}

template <typename F>
void with_log_small(int n, F&& f) {
  switch (n) {
    case 16: f(std::integral_constant<int, 4>{}); break;
    case 32: f(std::integral_constant<int, 5>{}); break;
    case 64: f(std::integral_constant<int, 6>{}); break;
    default: throw std::invalid_argument("solve in one workgroup: 16, 32 or 64 nodes an axis");
  }
}
template <typename T, typename F>
void with_small(const Geom& g, F&& f) {
  with_log_small(g.nx, [&](auto lx) {
    with_log_small(g.ny, [&](auto ly) { f(Small<T, decltype(lx)::value, decltype(ly)::value>{}, lx, ly); });
  });
}
void allow_lds(const void* fn, size_t lds) {
  if (lds > 65536)
    QSP_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
}

}  // namespace

template <typename T>
void launch_small_bxby(const Geom& g, const SrcBxBy<T>& s, const PCArgs<T>& pc, const ZeroJob& z,
                       const AxisTables<T>& tx, const AxisTables<T>& ty, const DevCounters* ctr,
                       hipStream_t st) {
  if (z.count != 2) throw std::invalid_argument("corrector solve: two trial planes to clear");
  with_small<T>(g, [&](auto sm, auto lx, auto ly) {
    using S = decltype(sm);
    constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
    if constexpr (small_grid(1 << LX, 1 << LY))
      hipLaunchKernelGGL((k_small_bxby<T, LX, LY>), dim3(2), dim3(S::BS), S::lds, st, g, s, pc, z, tx, ty, ctr);
    else
      throw std::invalid_argument("corrector solve: grid too large for one workgroup");
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_small_pez(const Geom& g, const SrcPEZ<T>& s, const RowInvArgs<T>& r, const ZeroJob& z,
                      const AxisTables<T>& tx, const AxisTables<T>& ty, hipStream_t st) {
  if (!r.guess.ctr || z.count < 0 || z.count > 8)
    throw std::invalid_argument("psi, Ez, Bz solve: bad guess or planes to clear");
  with_small<T>(g, [&](auto sm, auto lx, auto ly) {
    using S = decltype(sm);
    constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
    if constexpr (small_grid(1 << LX, 1 << LY))
      hipLaunchKernelGGL((k_small_pez<T, LX, LY>), dim3(4 + z.count), dim3(S::BS), S::lds, st, g, s, r, z, tx, ty);
    else
      throw std::invalid_argument("psi, Ez, Bz solve: grid too large for one workgroup");
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_small_nodes(const Geom& g, const T* src, T* dst, int nbatch, double shift,
                        const AxisTables<T>& tx, const AxisTables<T>& ty, hipStream_t st) {
  if (nbatch < 1) throw std::invalid_argument("solve in one workgroup: bad batch");
  with_small<T>(g, [&](auto sm, auto lx, auto ly) {
    using S = decltype(sm);
    constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
    allow_lds(reinterpret_cast<const void*>(&k_small_nodes<T, LX, LY>), S::lds);
    hipLaunchKernelGGL((k_small_nodes<T, LX, LY>), dim3(nbatch), dim3(S::BS), S::lds, st, src, dst, shift, tx, ty);
  });
  QSP_LAUNCH_CHECK();
}

#define QSP_INST(T)                                                                              \
  template void launch_small_bxby<T>(const Geom&, const SrcBxBy<T>&, const PCArgs<T>&,           \
                                     const ZeroJob&, const AxisTables<T>&, const AxisTables<T>&, \
                                     const DevCounters*, hipStream_t);                           \
  template void launch_small_pez<T>(const Geom&, const SrcPEZ<T>&, const RowInvArgs<T>&,         \
                                    const ZeroJob&, const AxisTables<T>&, const AxisTables<T>&,  \
                                    hipStream_t);                                                \
  template void launch_small_nodes<T>(const Geom&, const T*, T*, int, double,                    \
                                      const AxisTables<T>&, const AxisTables<T>&, hipStream_t);
QSP_INST(float)
QSP_INST(double)
#undef QSP_INST

}  // namespace qsp
