// Batched 2D Dirichlet Poisson / Helmholtz solve kernels and their launchers
// (fast Poisson solver of HiPACE++, arXiv:2109.10277 Sec. III.B).  The
// transform machinery and the per-block bodies live in dst_impl.hpp.
#include "dst_impl.hpp"

namespace qsp {

using namespace dst_detail;

// ---------------------------------------------------------------------------
// P1: sources + forward DST along x
// ---------------------------------------------------------------------------

// field ids of the psi / Ez / Bz batch
template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_src_fwd_pez(Geom g, SrcPEZ<T> a, AxisTables<T> tx) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  // neighbouring row blocks share the 128-byte lines of strip-ordered
  // planes: keep them on one XCD (one L2)
  const int j0 = xcd_strip(blockIdx.x, gridDim.x) * R;
  const int fld = blockIdx.y;   // 0 psi, 1 Ez, 2 Bz
  // psi: -(rho - Jz + ions); Ez: d_x Jx + d_y Jy; Bz: d_y Jx - d_x Jy
  const double ihx = fld == 1 ? 0.5 / g.hx : -0.5 / g.hx, ihy = 0.5 / g.hy;
  const double* __restrict__ ax = fld == 0 ? a.rho_mjz : (fld == 1 ? a.jx : a.jy);
  const double* __restrict__ ay = fld == 1 ? a.jy : a.jx;
  struct In {
    double e, w, n, s;
    __device__ void pin() {
      dst_detail::pin(e);
      dst_detail::pin(w);
      dst_detail::pin(n);
      dst_detail::pin(s);
    }
  };
  auto put = [&](int e, double s) {
    const int r = e >> LOGN, i = e & (n - 1);
    buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)] = static_cast<T>((i > 0 && j0 + r > 0) ? s : 0.0);
  };
  if (fld == 0) {
    struct Rho {
      double r;
      __device__ void pin() { dst_detail::pin(r); }
    };
    const bool ions = a.ionx != nullptr;
    for_row_batches<R, LOGN, 2 * src_batch<T, LOGN>(), Rho>(
        [&](int e, Rho& v) { v.r = load_at(ax, j0 * n + e); },
        [&](int, int e, const Rho& v) {
          put(e, -(v.r + (ions ? a.n0 * a.ionx[e & (n - 1)] * a.iony[j0 + (e >> LOGN)] : a.n0)));
        });
  } else {
    // neighbour indices are clamped so that every load is in bounds; values
    // outside the interior are replaced by selects
    for_row_batches<R, LOGN, src_batch<T, LOGN>(), In>(
        [&](int e, In& v) {
          const int i = e & (n - 1), j = j0 + (e >> LOGN);
          const int o = j * n + i;
          v.e = load_at(ax, i + 1 < n ? o + 1 : o);
          v.w = load_at(ax, i > 0 ? o - 1 : o);
          v.n = load_at(ay, j + 1 < g.ny ? o + n : o);
          v.s = load_at(ay, j > 0 ? o - n : o);
        },
        [&](int, int e, const In& v) {
          const int i = e & (n - 1), j = j0 + (e >> LOGN);
          put(e, ((i + 1 < n ? v.e : 0.0) - v.w) * ihx + ((j + 1 < g.ny ? v.n : 0.0) - v.s) * ihy);
        });
  }
  xf.commit();
  __syncthreads();
  block_dst<T, LOGN, true>(buf, ppitch, xf);
  rows_to_plane<T, R, LOGN>(g, j0, buf, ppitch, a.out + static_cast<size_t>(fld) * g.nx * g.ny);
}

template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_src_fwd_bxby(Geom g, SrcBxBy<T> a, AxisTables<T> tx, const DevCounters* ctr) {
  if (ctr->pc_done) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  src_bxby_block<T, LOGN>(g, a, tx, xcd_strip(blockIdx.x, gridDim.x), blockIdx.y, smem_raw);
}

// ---------------------------------------------------------------------------
// P2: column strip solve
// ---------------------------------------------------------------------------
template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, col_blocks_per_cu(LOGN, sizeof(T)))
k_col_solve(Geom g, ColArgs<T> a, AxisTables<T> ty, const double* __restrict__ lamx,
            const DevCounters* ctr) {
  if (a.honor_done && ctr->pc_done) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  col_block<T, LOGN>(g, a, ty, lamx, xcd_strip(blockIdx.x, gridDim.x), blockIdx.y, smem_raw);
  // the side job's stores come last (the memory counter the strip load waits
  // on also counts stores); the symmetric core's pass issues them itself,
  // before its transforms
  if constexpr (!sym_core(sizeof(T), 1 << LOGN))
    zero_job(a.zero, static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x,
             static_cast<size_t>(gridDim.x) * gridDim.y);
}

// ---------------------------------------------------------------------------
// P3: inverse DST along x with epilogues
// ---------------------------------------------------------------------------
template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_row_inv(Geom g, RowInvArgs<T> a, AxisTables<T> tx) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  const int j0 = xcd_strip(blockIdx.x, gridDim.x) * R;   // neighbours on one XCD
  const int fld = blockIdx.y;
  const size_t plane = static_cast<size_t>(g.nx) * g.ny;
  const size_t gstride = static_cast<size_t>(gridDim.x) * gridDim.y * kBlock;
  const size_t gi0 = (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
  GuessRegs<T> gr;
  RowFetch<T, R, LOGN> rows;
  rows.load(g, j0, a.in[fld]);
  if (a.guess.ctr) guess_load(a.guess, plane, gi0, gstride, gr);
  __builtin_amdgcn_sched_barrier(0);
  rows.put(g, buf, ppitch);
  xf.commit();
  if (a.guess.ctr) {   // its stores drain under the transform
    if (gi0 == 0) {
      a.guess.ctr->pc_done = 0u;
      a.guess.ctr->pc_iters = 0u;
      a.guess.ctr->pc_resid = 0.0;
    }
    guess_store(a.guess, plane, gi0, gstride, gr);
    for (size_t i0 = gi0 + kGuess * gstride; i0 < plane; i0 += kGuess * gstride) {
      guess_load(a.guess, plane, i0, gstride, gr);
      guess_store(a.guess, plane, i0, gstride, gr);
    }
  }
  __syncthreads();
  block_dst<T, LOGN, false>(buf, ppitch, xf);
  T* out = a.out[fld];
  T* out_dx = a.out_dx[fld];
  const T mihx = static_cast<T>(-0.5 / g.hx);
  // tested once: per element the loop stays rolled (21.7 against 20.2 us at
  // 1024^2 in FP32)
  auto put = [&](auto with_dx) {
    for_row_elems<R, LOGN>([&](int e) {
      const int r = e >> LOGN, i = e & (n - 1);
      const int j = j0 + r;
      const T* row = buf + RowLay<T, LOGN>::rpos(n, ppitch, r, 0);
      const T u = row[RowLay<T, LOGN>::ridx(i)];
      store_at(out, j * n + i, j > 0 ? u : T(0));
      if constexpr (decltype(with_dx)::value) {
        const T ue = row[RowLay<T, LOGN>::ridx(i + 1 < n ? i + 1 : i)], uw = row[RowLay<T, LOGN>::ridx(i > 0 ? i - 1 : 0)];
        const T d = mihx * ((i + 1 < n ? ue : T(0)) - uw);
        store_at(out_dx, j * n + i, (i > 0 && j > 0) ? d : T(0));
      }
    });
  };
  if (out_dx)
    put(std::true_type{});
  else
    put(std::false_type{});
}

// First and last pass of a batched solve on the caller's node arrays
// ([ny+1][nx+1], row j at j (nx + 1)): OUT = false reads the sources straight
// into the rows (boundary nodes taken as zero) and writes an intermediate
// plane, OUT = true reads one and writes the solution with its zero boundary.
// Both ends are bound by latency and launches: as separate layout copies they
// took 4.6 us a plane, 27 of the 66 us of a batch of three at 1024^2 in FP32.
template <typename T, int LOGN, bool OUT>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_row_nodes(Geom g, NodeRowArgs<T> a, AxisTables<T> tx) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  const int j0 = xcd_strip(blockIdx.x, gridDim.x) * R;
  const int b = blockIdx.y;
  const size_t plane = static_cast<size_t>(n) * g.ny;
  const size_t nodes = static_cast<size_t>(n + 1) * (g.ny + 1);
  if constexpr (!OUT) {
    const T* __restrict__ src = a.nodes_in + b * nodes;
    for_row_elems<R, LOGN>([&](int e) {
      const int r = e >> LOGN, i = e & (n - 1);
      const int j = j0 + r;
      const T v = load_at(src, j * (n + 1) + i);
      buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)] = i > 0 && j > 0 ? v : T(0);
    });
  } else {
    RowFetch<T, R, LOGN> rows;
    rows.load(g, j0, a.plane + b * plane);
    __builtin_amdgcn_sched_barrier(0);
    rows.put(g, buf, ppitch);
  }
  xf.commit();
  __syncthreads();
  block_dst<T, LOGN, !OUT>(buf, ppitch, xf);
  if constexpr (!OUT) {
    rows_to_plane<T, R, LOGN>(g, j0, buf, ppitch, a.plane + b * plane);
  } else {
    T* __restrict__ dst = a.nodes_out + b * nodes;
    for_row_elems<R, LOGN>([&](int e) {
      const int r = e >> LOGN, i = e & (n - 1);
      const int j = j0 + r;
      const T v = buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)];
      store_at(dst, j * (n + 1) + i, j > 0 ? v : T(0));
    });
    if (static_cast<int>(threadIdx.x) < R) dst[(j0 + static_cast<int>(threadIdx.x)) * (n + 1) + n] = T(0);
    if (j0 + R == g.ny)
      for (int i = threadIdx.x; i <= n; i += kBlock) dst[g.ny * (n + 1) + i] = T(0);
  }
}

template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_row_inv_pc(Geom g, PCArgs<T> a, AxisTables<T> tx, DevCounters* ctr) {
  if (ctr->pc_done) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  row_inv_pc_block<T, LOGN>(g, a, tx, xcd_strip(blockIdx.x, gridDim.x), blockIdx.y, smem_raw);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Workgroups above 64 KiB of LDS (large grids, FP64) opt in explicitly; gfx950
// offers 160 KiB per workgroup.
static void allow_lds(const void* fn, size_t lds) {
  if (lds > 65536)
    QSP_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(lds)));
}

template <typename T>
void launch_src_fwd_pez(const Geom& g, const SrcPEZ<T>& a, const AxisTables<T>& tx,
                        hipStream_t st) {
  const int R = pass_rows<T>(g.nx);
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    allow_lds(reinterpret_cast<const void*>(&k_src_fwd_pez<T, E>), lds);
    hipLaunchKernelGGL((k_src_fwd_pez<T, E>), dim3(g.ny / R, 3), dim3(kBlock), lds, st, g, a, tx);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_src_fwd_bxby(const Geom& g, const SrcBxBy<T>& a, const AxisTables<T>& tx,
                         const DevCounters* ctr, hipStream_t st) {
  const int R = pass_rows<T>(g.nx);
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    allow_lds(reinterpret_cast<const void*>(&k_src_fwd_bxby<T, E>), lds);
    hipLaunchKernelGGL((k_src_fwd_bxby<T, E>), dim3(g.ny / R, 2), dim3(kBlock), lds, st, g, a, tx,
                       ctr);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_col_solve(const Geom& g, const ColArgs<T>& a, int nfield, const AxisTables<T>& ty,
                      const double* lamx, const DevCounters* ctr, hipStream_t st) {
  const int W = a.w;
  if (W != pass_cols<T>(g.ny) || nfield < 1 || nfield > 4)
    throw std::invalid_argument("column pass: bad strip width or field count");
  if (g.strip && W != 4)   // a strip of the intermediate planes is 4 columns
    throw std::invalid_argument("column pass: strip-ordered planes need strips of 4 columns");
  const size_t lds = pass_lds<T>(W, g.ny);
  with_logn(g.ny, [&](auto e) {
    constexpr int E = decltype(e)::value;
    allow_lds(reinterpret_cast<const void*>(&k_col_solve<T, E>), lds);
    hipLaunchKernelGGL((k_col_solve<T, E>), dim3(g.nx / W, nfield), dim3(kBlock), lds, st, g, a,
                       ty, lamx, ctr);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_row_inv(const Geom& g, const RowInvArgs<T>& a, int nfield, const AxisTables<T>& tx,
                    hipStream_t st) {
  const int R = pass_rows<T>(g.nx);
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    allow_lds(reinterpret_cast<const void*>(&k_row_inv<T, E>), lds);
    hipLaunchKernelGGL((k_row_inv<T, E>), dim3(g.ny / R, nfield), dim3(kBlock), lds, st, g, a, tx);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_row_nodes(const Geom& g, const NodeRowArgs<T>& a, bool out, int nbatch,
                      const AxisTables<T>& tx, hipStream_t st) {
  const int R = pass_rows<T>(g.nx);
  if (nbatch < 1 || nbatch > 4 || !a.plane || (out ? !a.nodes_out : !a.nodes_in))
    throw std::invalid_argument("node row pass: bad planes or batch");
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    const dim3 grid(g.ny / R, nbatch);
    if (out) {
      allow_lds(reinterpret_cast<const void*>(&k_row_nodes<T, E, true>), lds);
      hipLaunchKernelGGL((k_row_nodes<T, E, true>), grid, dim3(kBlock), lds, st, g, a, tx);
    } else {
      allow_lds(reinterpret_cast<const void*>(&k_row_nodes<T, E, false>), lds);
      hipLaunchKernelGGL((k_row_nodes<T, E, false>), grid, dim3(kBlock), lds, st, g, a, tx);
    }
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_row_inv_pc(const Geom& g, const PCArgs<T>& a, const AxisTables<T>& tx,
                       DevCounters* ctr, hipStream_t st) {
  const int R = pass_rows<T>(g.nx);
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    allow_lds(reinterpret_cast<const void*>(&k_row_inv_pc<T, E>), lds);
    hipLaunchKernelGGL((k_row_inv_pc<T, E>), dim3(g.ny / R, 2), dim3(kBlock), lds, st, g, a, tx,
                       ctr);
  });
  QSP_LAUNCH_CHECK();
}

int pc_partial_count(const Geom& g) {
  return small_grid(g.nx, g.ny) ? 2 : 2 * (g.ny / g.rr);   // one record a field, or a row block
}

template <typename T>
int col_width(const Geom& g) {
  return pass_cols<T>(g.ny);
}
template int col_width<float>(const Geom&);
template int col_width<double>(const Geom&);
template <typename T>
int row_rows(int nx) {
  return pass_rows<T>(nx);
}
template int row_rows<float>(int);
template int row_rows<double>(int);

#define QSP_INST(T)                                                                       \
  template void launch_src_fwd_pez<T>(const Geom&, const SrcPEZ<T>&, const AxisTables<T>&, \
                                      hipStream_t);                                        \
  template void launch_src_fwd_bxby<T>(const Geom&, const SrcBxBy<T>&,                     \
                                       const AxisTables<T>&, const DevCounters*,           \
                                       hipStream_t);                                       \
  template void launch_col_solve<T>(const Geom&, const ColArgs<T>&, int,                   \
                                    const AxisTables<T>&, const double*,                   \
                                    const DevCounters*, hipStream_t);                      \
  template void launch_row_inv<T>(const Geom&, const RowInvArgs<T>&, int,                  \
                                  const AxisTables<T>&, hipStream_t);                      \
  template void launch_row_nodes<T>(const Geom&, const NodeRowArgs<T>&, bool, int,         \
                                    const AxisTables<T>&, hipStream_t);                    \
  template void launch_row_inv_pc<T>(const Geom&, const PCArgs<T>&, const AxisTables<T>&,  \
                                     DevCounters*, hipStream_t);
QSP_INST(float)
QSP_INST(double)
#undef QSP_INST

}  // namespace qsp
