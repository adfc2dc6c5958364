// Adjoint (reverse-mode) kernels of the slice loop.  Every kernel is the
// transpose of a forward step of the HiPACE++ slice routine (arXiv:2109.10277
// Sec. II, III.B) as the forward kernels discretise it:
//   * field gather (shape S of order 1-3)
//                                   -> FP64 scatter of the gathered adjoints
//                                      plus grad-S position terms;
//   * deposit (shape S)             -> gather of the adjoint planes with S and
//                                      grad S;
//   * pusher right-hand side        -> its Jacobian, transposed;
//   * Adams-Bashforth step          -> ring of the step adjoints of the last
//                                      four slices (slot j mod 4);
//   * (lap - s)^-1, centred d/dx    -> the same solves, D^T = -D.
// Positions are the displacements xi (cell units) of the forward kernels, so
// the position adjoints are per cell.  Particles the step absorbs, dead
// particles and floored 1+Psi are locally constant.
#include "common.hpp"
#include "dst_impl.hpp"
#include "kernels.hpp"
#include "partials.hpp"
#include "push_tile.hpp"
#include "shape.hpp"

namespace qsp {

using namespace dst_detail;

namespace {

__device__ inline void gadd(double* p, double v) { unsafeAtomicAdd(p, v); }

// One axis of a particle's stencil: lowest node b, fraction d, clamped node
// indices, and the shape weights and their slopes (per cell) in precision R,
// zero on the nodes that are not stored.
template <int O, typename R>
struct Axis {
  int b;
  R d;
  int idx[O + 1];
  R w[O + 1], g[O + 1];
};

template <int O, typename R>
__device__ inline Axis<O, R> make_axis(int b, R d, int n) {
  Axis<O, R> A;
  A.b = b;
  A.d = d;
  bool ok[O + 1];
  shape::weights<O>(d, A.w);
  shape::weight_slopes<O>(d, A.g);
  shape::axis_nodes<O>(b, n, A.idx, ok);
#pragma unroll
  for (int q = 0; q <= O; ++q) {
    A.w[q] = ok[q] ? A.w[q] : R(0);
    A.g[q] = ok[q] ? A.g[q] : R(0);
  }
  return A;
}

template <int O, typename T>
__device__ inline Axis<O, T> locate_axis(int c0, T t, int n) {
  int b;
  const T d = shape::locate<O>(c0, t, n, b);
  return make_axis<O, T>(b, d, n);
}

// value and position gradient (per cell) of the shape interpolant of F
template <int O, typename T, typename R>
__device__ inline void interp(const T* __restrict__ F, const Axis<O, R>& X, const Axis<O, R>& Y,
                              int nx, R& v, R& gx, R& gy) {
  v = R(0);
  gx = R(0);
  gy = R(0);
#pragma unroll
  for (int b = 0; b <= O; ++b) {
    const T* row = F + static_cast<size_t>(Y.idx[b]) * nx;
    R rv = R(0), rg = R(0);
#pragma unroll
    for (int a = 0; a <= O; ++a) {
      const R f = static_cast<R>(row[X.idx[a]]);
      rv += X.w[a] * f;
      rg += X.g[a] * f;
    }
    v += Y.w[b] * rv;
    gx += Y.w[b] * rg;
    gy += Y.g[b] * rv;
  }
}

}  // namespace

// Deposit transpose of the trial currents: from the gathered adjoints of
// Jx~ (= +lsb_y / 2dz) and Jy~ (= -lsb_x / 2dz) at the trial position, the
// adjoints of the trial state (offsets, u, Psi).
template <typename T, int O>
__device__ __forceinline__ void trial_deposit_adjoint(const AdjPushArgs<T>& a, int ci0, int cj0,
                                                      T fx0, T fy0, T xn, T en, T tux, T tuy,
                                                      T psin, T w, int nx, int ny, T (&v)[5]) {
  const Axis<O, T> TX = locate_axis<O>(ci0, fx0 + xn, nx);
  const Axis<O, T> TY = locate_axis<O>(cj0, fy0 + en, ny);
  T gjx, gjx_x, gjx_y, gjy, gjy_x, gjy_y;
  interp(a.lsb_y, TX, TY, nx, gjx, gjx_x, gjx_y);
  interp(a.lsb_x, TX, TY, nx, gjy, gjy_x, gjy_y);
  const T s2 = static_cast<T>(a.inv2dz);
  gjx *= s2; gjx_x *= s2; gjx_y *= s2;
  gjy *= -s2; gjy_x *= -s2; gjy_y *= -s2;
  const T floor_d = static_cast<T>(a.psi_floor);
  const T tdraw = T(1) + psin;
  const bool tun = !(tdraw < floor_d);
  const T tid = T(1) / (tun ? tdraw : floor_d);
  const T qn = -w;
  const T vjx = qn * tux * tid, vjy = qn * tuy * tid;
  v[0] = vjx * gjx_x + vjy * gjy_x;
  v[1] = vjx * gjx_y + vjy * gjy_y;
  v[2] = qn * tid * gjx;
  v[3] = qn * tid * gjy;
  v[4] = tun ? (-qn * tux * tid * tid * gjx - qn * tuy * tid * tid * gjy) : T(0);
}

// Transpose of one real (MODE 0) or trial (MODE 1) push from the taped
// state of slice k.  Real: lam_y holds the adjoint of the pushed state on
// entry and that of the slice-k state (push part) on exit.  Trial: the
// adjoint of the trial state comes from the trial-current adjoints gathered
// at the recorded trial position and is added to lam_y.
//
// The Adams-Bashforth history is transposed through a ring of the last four
// slices' step adjoints: slot j mod 4 holds the adjoint Lambda_j of the
// states pushed from slice j (real push and trials), and the adjoint that
// f_k collects from the later steps is -dz sum_m b_m Lambda_{k+m}.  So the
// real push reads the ring (20 values) and stores its own slot (5), the
// trial adds to that slot, and neither needs the forward history: whether
// the particle stayed in the box, and its trial state, come from the trial
// record.  Bound by HBM: with the history read and every slot of the ring
// read, modified and written in both pushes (76 and 83 values a particle
// instead of 43 and 39) they took 364 and 431 us at 1024^2, 4 ppc, FP32.
// Every value of a particle is fetched at once (AdjPushLoad), in front of the
// histogram's clear: the compiler keeps each read-modify-write in its place
// otherwise, ten memory round trips in a row (1024^2, 4 ppc, FP32: trial 226 ->
// 168 us, real 194 -> 173, later trials 97 -> 79).
template <typename T, int MODE>
struct AdjPushLoad {
  T w, fac, y[5], ly[5];
  T ring[MODE == 0 ? 4 : 1][5];   // real: Lambda_{k+m}, m = 1..4; trial: Lambda_k
  T rec[5], acc[7];               // trial: position and momentum, Psi; later iterations' sums
  __device__ __forceinline__ void load(const Lattice& L, const AdjPushArgs<T>& a, unsigned int p) {
    const size_t np = static_cast<size_t>(L.np), np5 = 5 * np;
    w = load_at(a.p.w, p);
    y[0] = load_at(a.p.xi_x, p);
    y[1] = load_at(a.p.xi_y, p);
    y[2] = load_at(a.p.ux, p);
    y[3] = load_at(a.p.uy, p);
    y[4] = load_at(a.p.psi, p);
    const T* q = a.rec;
#pragma unroll
    for (int c = 0; c < 6; ++c, q += np) {
      if (c == 4)
        fac = load_at(q, p);   // 0: absorbed by the step
      else if constexpr (MODE == 1)
        rec[c < 4 ? c : 4] = load_at(q, p);
    }
    q = a.lam_y;
#pragma unroll
    for (int c = 0; c < 5; ++c, q += np) ly[c] = load_at(q, p);
#pragma unroll
    for (int m = 0; m < (MODE == 0 ? 4 : 1); ++m) {
      q = a.lam_ring + static_cast<size_t>((a.k + (MODE == 0 ? m + 1 : 0)) & 3) * np5;
#pragma unroll
      for (int c = 0; c < 5; ++c, q += np) ring[m][c] = load_at(q, p);
    }
    if (MODE == 1 && a.acc) {
      q = a.acc;
#pragma unroll
      for (int c = 0; c < 7; ++c, q += np) acc[c] = load_at(q, p);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

template <typename T, int MODE, int O, typename Scatter>
__device__ __forceinline__ void adj_push_one(const Geom& g, const Lattice& L,
                                             const AdjPushArgs<T>& a, AdjPushLoad<T, MODE>& in,
                                             int I, int J, Scatter&& scat) {
  const size_t np = static_cast<size_t>(L.np);
  const unsigned int p = static_cast<unsigned int>(J) * static_cast<unsigned int>(L.nX) +
                         static_cast<unsigned int>(I);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    push_detail::pin(in.y[c]);
    push_detail::pin(in.ly[c]);
  }
  const T w = in.w, fac = in.fac;
  const T (&y)[5] = in.y;
  const T dz = static_cast<T>(a.dzeta);
  const T b[5] = {T(kAB5[0]), T(kAB5[1]), T(kAB5[2]), T(kAB5[3]), T(kAB5[4])};
  T* ly = a.lam_y;
  T* own = a.lam_ring + static_cast<size_t>(a.k & 3) * 5 * np;   // Lambda_k (and _{k+4} before)
  const bool moved = fac != T(0);
  T lnew[5] = {0, 0, 0, 0, 0};
  T lf[5] = {0, 0, 0, 0, 0};
  T lf_own[2] = {0, 0};   // trial: lf[2], lf[3] of this iteration's deposit alone
  if (MODE == 0) {
    constexpr int M = MODE == 0 ? 4 : 1;   // rows of in.ring
#pragma unroll
    for (int c = 0; c < 5; ++c) lnew[c] = in.ly[c];
    if (w == T(0)) return;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      if (!moved) lnew[c] = T(0);
      const T sum = b[0] * lnew[c] + (b[1] * in.ring[0][c] + b[2] * in.ring[1 % M][c] +
                                      b[3] * in.ring[2 % M][c] + b[4] * in.ring[3 % M][c]);
      lf[c] = moved ? -dz * sum : T(0);
      store_at(own + c * np, p, lnew[c]);
    }
    if (!moved) {
#pragma unroll
      for (int c = 0; c < 5; ++c) store_at(ly + c * np, p, T(0));
      return;
    }
  } else {
    if (w == T(0) || !moved) return;   // nothing deposited by any iteration
  }
  const int nx = g.nx, ny = g.ny;
  const int lpx = 31 - __clz(L.ppc_x), lpy = 31 - __clz(L.ppc_y);
  const int ci0 = I >> lpx, cj0 = J >> lpy;
  const T fx0 = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
  const T fy0 = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
  const T inv_hx = static_cast<T>(1.0 / a.hx), inv_hy = static_cast<T>(1.0 / a.hy);
  const T floor_d = static_cast<T>(a.psi_floor);
  // gather with gradients at the current position
  const Axis<O, T> X = locate_axis<O>(ci0, fx0 + y[0], nx);
  const Axis<O, T> Y = locate_axis<O>(cj0, fy0 + y[1], ny);
  T v[6], gx[6], gy[6];
  const T* F[6] = {a.f.exmby, a.f.eypbx, a.f.ez, a.f.bx, a.f.by, a.f.bz};
#pragma unroll
  for (int c = 0; c < 6; ++c) interp(F[c], X, Y, nx, v[c], gx[c], gy[c]);
  const T e1 = v[0], e2 = v[1], bx = v[3], by = v[4], bz = v[5];
  const T ux = y[2], uy = y[3];
  const T draw = T(1) + y[4];
  const bool unclamped = !(draw < floor_d);
  const T d = unclamped ? draw : floor_d;
  const T id = T(1) / d;
  const T u2 = T(1) + ux * ux + uy * uy;
  const T gam = (T(1) + ux * ux + uy * uy + d * d) * T(0.5) * id;
  const T G = gam * id;                              // gamma / D
  if (MODE == 1) {
    const T kick = dz * b[0];
    trial_deposit_adjoint<T, O>(a, ci0, cj0, fx0, fy0, in.rec[0], in.rec[1], in.rec[2] - kick * by,
                                in.rec[3] + kick * bx, in.rec[4], w, nx, ny, lnew);
    // this iteration's own Bx, By terms use its own deposit adjoint only;
    // the later iterations' sums join everything they share with it
#pragma unroll
    for (int c = 2; c < 4; ++c) lf_own[c - 2] = -dz * b[0] * lnew[c];
    if (a.acc)
#pragma unroll
      for (int c = 0; c < 5; ++c) lnew[c] += in.acc[c];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      lf[c] = -dz * b[0] * lnew[c];
      store_at(own + c * np, p, in.ring[0][c] + lnew[c]);
    }
  }
  // the identity part of the step
  T lam[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) lam[c] = lnew[c];
  // right-hand side transposed
  const T id2 = id * id;
  T lux = -lf[0] * id * inv_hx + lf[2] * (ux * id2) * e1 + lf[3] * ((ux * id2) * e2 - bz * id) + lf[4] * e1 * id;
  T luy = -lf[1] * id * inv_hy + lf[2] * ((uy * id2) * e1 + bz * id) + lf[3] * (uy * id2) * e2 + lf[4] * e2 * id;
  T ld = lf[0] * ux * id2 * inv_hx + lf[1] * uy * id2 * inv_hy +
         lf[2] * (-u2 * id2 * id * e1 - bz * uy * id2) + lf[3] * (-u2 * id2 * id * e2 + bz * ux * id2) +
         lf[4] * (-(ux * e1 + uy * e2) * id2);
  lam[2] += lux;
  lam[3] += luy;
  if (unclamped) lam[4] += ld;
  T lg[6];
  lg[0] = lf[2] * G + lf[4] * ux * id;
  lg[1] = lf[3] * G + lf[4] * uy * id;
  lg[2] = -lf[4];
  lg[3] = MODE == 0 ? -lf[3] : -lf_own[1];
  lg[4] = MODE == 0 ? lf[2] : lf_own[0];
  lg[5] = lf[2] * uy * id - lf[3] * ux * id;
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    lam[0] += lg[c] * gx[c];
    lam[1] += lg[c] * gy[c];
    scat(c, X, Y, static_cast<double>(lg[c]));
  }
  if (MODE == 1 && a.acc) {   // the later iterations' own Bx, By position terms
    lam[0] += in.acc[5];
    lam[1] += in.acc[6];
  }
  if (MODE == 0) {
#pragma unroll
    for (int c = 0; c < 5; ++c) store_at(ly + c * np, p, lam[c]);
  } else {
#pragma unroll
    for (int c = 0; c < 5; ++c) store_at(ly + c * np, p, in.ly[c] + lam[c]);
  }
}

// One workgroup per lattice tile (the tiles of the forward push): the
// transposed gathers of the six fields accumulate in FP64 LDS histograms of
// the tile's cells plus a halo and reach the global planes with one atomic
// per non-zero node; stencils outside the histogram go straight to global
// atomics.
template <typename T, int MODE, int O>
__global__ void __launch_bounds__(kBlock) k_adj_push(Geom g, Lattice L, AdjPushArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* tile = reinterpret_cast<double*>(smem_raw);
  const push_detail::TileShape ts = push_detail::tile_shape(L, a.tile_rows, a.tile_halo);
  const int ntile = ts.nw * ts.nh;
  const int nx = g.nx, ny = g.ny;
  const int I0 = push_detail::tile_column(false) * ts.tx, J0 = blockIdx.y * ts.ty;
  AdjPushLoad<T, MODE> in;
  in.load(L, a, push_detail::tile_particle(L, ts, I0, J0, static_cast<int>(threadIdx.x)));
  for (int e = threadIdx.x; e < 6 * ntile; e += kBlock) tile[e] = 0.0;
  __syncthreads();
  const int ox = (I0 >> ts.lpx) - ts.halo, oy = (J0 >> ts.lpy) - ts.halo;
  auto scat = [&](int c, const Axis<O, T>& X, const Axis<O, T>& Y, double v) {
    if (v == 0.0) return;
    double sx[O + 1], sy[O + 1];
    shape::weights<O>(static_cast<double>(X.d), sx);
    shape::weights<O>(static_cast<double>(Y.d), sy);
    const int li = X.b - ox, lj = Y.b - oy;
    if (li >= 0 && li + O < ts.nw && lj >= 0 && lj + O < ts.nh) {
      double* t = tile + c * ntile + lj * ts.nw + li;
#pragma unroll
      for (int qb = 0; qb <= O; ++qb)
#pragma unroll
        for (int qa = 0; qa <= O; ++qa) push_detail::lds_add(t + qb * ts.nw + qa, v * (sx[qa] * sy[qb]));
    } else {
#pragma unroll
      for (int qb = 0; qb <= O; ++qb) {
        const int j = Y.b + qb;
#pragma unroll
        for (int qa = 0; qa <= O; ++qa) {
          const int i = X.b + qa;
          if (i >= 1 && i < nx && j >= 1 && j < ny)
            gadd(a.lam_F[c] + static_cast<size_t>(j) * nx + i, v * (sx[qa] * sy[qb]));
        }
      }
    }
  };
  for (int e = threadIdx.x; e < ts.tx * ts.ty; e += kBlock) {
    if (e >= kBlock) in.load(L, a, push_detail::tile_particle(L, ts, I0, J0, e));
    adj_push_one<T, MODE, O>(g, L, a, in, I0 + (e & (ts.tx - 1)), J0 + (e >> ts.ltx), scat);
  }
  __syncthreads();
  push_detail::flush_tile<6>(a.lam_F, tile, ts, ox, oy, nx, ny);
}

// Transpose of a later predictor-corrector trial push (iteration m >= 1),
// which the forward computes from the slice's trial record: the deposit of
// Jx, Jy at the recorded position with u = u0 - dz b0 (By, -Bx)(x_k).  Its
// Bx, By adjoints are scattered at the slice-k position (the B cotangent of
// iteration m); the adjoints of the recorded quantities, which the first
// trial push's transpose carries back to the state, history and E fields,
// are summed per particle into acc (with the slice-k position terms of this
// iteration's own Bx, By gradients).
template <typename T>
struct AdjLaterLoad {   // fetched at once, like AdjPushLoad
  T w, xk, ek, rec[6], acc[7];
  __device__ __forceinline__ void load(const Lattice& L, const AdjPushArgs<T>& a, unsigned int p) {
    const size_t np = static_cast<size_t>(L.np);
    w = load_at(a.p.w, p);
    xk = load_at(a.p.xi_x, p);
    ek = load_at(a.p.xi_y, p);
    const T* q = a.rec;
#pragma unroll
    for (int c = 0; c < 6; ++c, q += np) rec[c] = load_at(q, p);
    if (a.acc_mode != 1) {
      q = a.acc;
#pragma unroll
      for (int c = 0; c < 7; ++c, q += np) acc[c] = load_at(q, p);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

template <typename T, int O, typename Scatter>
__device__ __forceinline__ void adj_trial_later_one(const Geom& g, const Lattice& L,
                                                    const AdjPushArgs<T>& a, AdjLaterLoad<T>& in,
                                                    int I, int J, Scatter&& scat) {
  const size_t np = static_cast<size_t>(L.np);
  const unsigned int p = static_cast<unsigned int>(J) * static_cast<unsigned int>(L.nX) +
                         static_cast<unsigned int>(I);
  T* acc = a.acc;
  const bool store = a.acc_mode == 1;
  push_detail::pin(in.xk);
  push_detail::pin(in.ek);
#pragma unroll
  for (int c = 0; c < 6; ++c) push_detail::pin(in.rec[c]);
  const T fac = in.rec[4];
  if (fac == T(0)) {   // dead, or absorbed by the step: nothing deposited
    if (store)
#pragma unroll
      for (int c = 0; c < 7; ++c) store_at(acc + c * np, p, T(0));
    return;
  }
  const T w = in.w;
  const T xk = in.xk, ek = in.ek;
  const T xn = in.rec[0], en = in.rec[1], cx = in.rec[2], cy = in.rec[3];
  const T psin = in.rec[5];
  const int nx = g.nx, ny = g.ny;
  const int lpx = 31 - __clz(L.ppc_x), lpy = 31 - __clz(L.ppc_y);
  const int ci0 = I >> lpx, cj0 = J >> lpy;
  const T fx0 = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
  const T fy0 = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
  const T dz = static_cast<T>(a.dzeta);
  const T b0 = T(kAB5[0]);
  // this iteration's Bx, By at the slice-k position, with gradients
  const Axis<O, T> X = locate_axis<O>(ci0, fx0 + xk, nx);
  const Axis<O, T> Y = locate_axis<O>(cj0, fy0 + ek, ny);
  T bx, bx_x, bx_y, by, by_x, by_y;
  interp(a.f.bx, X, Y, nx, bx, bx_x, bx_y);
  interp(a.f.by, X, Y, nx, by, by_x, by_y);
  const T kick = dz * b0;
  T v[7];
  {
    T d5[5];
    trial_deposit_adjoint<T, O>(a, ci0, cj0, fx0, fy0, xn, en, cx - kick * by, cy + kick * bx, psin,
                                w, nx, ny, d5);
#pragma unroll
    for (int c = 0; c < 5; ++c) v[c] = d5[c];
  }
  // f_x carries +By, f_y -Bx, each times -dz b0 in the step
  const T lgbx = dz * b0 * v[3], lgby = -dz * b0 * v[2];
  scat(0, X, Y, static_cast<double>(lgbx));
  scat(1, X, Y, static_cast<double>(lgby));
  v[5] = lgbx * bx_x + lgby * by_x;
  v[6] = lgbx * bx_y + lgby * by_y;
#pragma unroll
  for (int c = 0; c < 7; ++c) store_at(acc + c * np, p, store ? v[c] : in.acc[c] + v[c]);
}

// Tiles as in k_adj_push; two LDS histograms (Bx, By adjoints of the
// iteration, lam_F[3] and lam_F[4]).
template <typename T, int O>
__global__ void __launch_bounds__(kBlock) k_adj_trial_later(Geom g, Lattice L, AdjPushArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* tile = reinterpret_cast<double*>(smem_raw);
  const push_detail::TileShape ts = push_detail::tile_shape(L, a.tile_rows, a.tile_halo);
  const int ntile = ts.nw * ts.nh;
  const int nx = g.nx, ny = g.ny;
  const int I0 = push_detail::tile_column(false) * ts.tx, J0 = blockIdx.y * ts.ty;
  AdjLaterLoad<T> in;
  in.load(L, a, push_detail::tile_particle(L, ts, I0, J0, static_cast<int>(threadIdx.x)));
  for (int e = threadIdx.x; e < 2 * ntile; e += kBlock) tile[e] = 0.0;
  __syncthreads();
  const int ox = (I0 >> ts.lpx) - ts.halo, oy = (J0 >> ts.lpy) - ts.halo;
  auto scat = [&](int c, const Axis<O, T>& X, const Axis<O, T>& Y, double v) {
    if (v == 0.0) return;
    double sx[O + 1], sy[O + 1];
    shape::weights<O>(static_cast<double>(X.d), sx);
    shape::weights<O>(static_cast<double>(Y.d), sy);
    const int li = X.b - ox, lj = Y.b - oy;
    if (li >= 0 && li + O < ts.nw && lj >= 0 && lj + O < ts.nh) {
      double* t = tile + c * ntile + lj * ts.nw + li;
#pragma unroll
      for (int qb = 0; qb <= O; ++qb)
#pragma unroll
        for (int qa = 0; qa <= O; ++qa) push_detail::lds_add(t + qb * ts.nw + qa, v * (sx[qa] * sy[qb]));
    } else {
#pragma unroll
      for (int qb = 0; qb <= O; ++qb) {
        const int j = Y.b + qb;
#pragma unroll
        for (int qa = 0; qa <= O; ++qa) {
          const int i = X.b + qa;
          if (i >= 1 && i < nx && j >= 1 && j < ny)
            gadd(a.lam_F[3 + c] + static_cast<size_t>(j) * nx + i, v * (sx[qa] * sy[qb]));
        }
      }
    }
  };
  for (int e = threadIdx.x; e < ts.tx * ts.ty; e += kBlock) {
    if (e >= kBlock) in.load(L, a, push_detail::tile_particle(L, ts, I0, J0, e));
    adj_trial_later_one<T, O>(g, L, a, in, I0 + (e & (ts.tx - 1)), J0 + (e >> ts.ltx), scat);
  }
  __syncthreads();
  push_detail::flush_tile<2>(a.lam_F + 3, tile, ts, ox, oy, nx, ny);
}

// Transpose of the deposit at the slice-k state: gathers the adjoints of
// rho-Jz, Jx, Jy, Jz (FP64 planes) with S and grad S.
template <typename T, int O>
__global__ void __launch_bounds__(kBlock) k_adj_deposit(Geom g, Lattice L, AdjDepArgs<T> a) {
  if (blockIdx.x == 0) {
    // the beam-parameter gradient of the slice from the grid kernel's partial
    // records (3 x 4096 atomics to three addresses took 90 of its 107 us)
    double t[3];
    partials::sum<3>(a.part, a.part_n, t);
    if (threadIdx.x == 0) {
      a.grad_amp[a.k] = -t[0];
      a.grad_sigma[0] += -a.amp * t[1];
      a.grad_sigma[1] += -a.amp * t[2];
    }
  }
  const size_t np = static_cast<size_t>(L.np);
  const unsigned int p = blockIdx.x * static_cast<unsigned int>(kBlock) + threadIdx.x;   // np < 2^30
  if (p >= np) return;
  T w = load_at(a.p.w, p);
  T xi = load_at(a.p.xi_x, p), eta = load_at(a.p.xi_y, p);
  T ux = load_at(a.p.ux, p), uy = load_at(a.p.uy, p), psi = load_at(a.p.psi, p);
  T ly[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) ly[c] = load_at(static_cast<const T*>(a.lam_y) + c * np, p);
  __builtin_amdgcn_sched_barrier(0);
  push_detail::pin(xi);
  push_detail::pin(eta);
#pragma unroll
  for (int c = 0; c < 5; ++c) push_detail::pin(ly[c]);
  if (w == T(0)) return;
  const int nx = g.nx, ny = g.ny;
  const int I = static_cast<int>(p & static_cast<unsigned int>(L.nX - 1)), J = static_cast<int>(p >> (31 - __clz(L.nX)));
  const int lpx = 31 - __clz(L.ppc_x), lpy = 31 - __clz(L.ppc_y);
  const T fx0 = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
  const T fy0 = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
  int bi, bj;
  const T dx = shape::locate<O>(I >> lpx, fx0 + xi, nx, bi);
  const T dy = shape::locate<O>(J >> lpy, fy0 + eta, ny, bj);
  const Axis<O, double> X = make_axis<O, double>(bi, static_cast<double>(dx), nx);
  const Axis<O, double> Y = make_axis<O, double>(bj, static_cast<double>(dy), ny);
  const T floor_d = static_cast<T>(a.psi_floor);
  const T draw = T(1) + psi;
  const bool un = !(draw < floor_d);
  const T d = un ? draw : floor_d;
  const T id = T(1) / d;
  const T u2 = T(1) + ux * ux + uy * uy;
  const T qn = -w;
  const T val[4] = {qn, qn * ux * id, qn * uy * id, qn * (u2 * T(0.5) * id * id - T(0.5))};
  const T dux[4] = {T(0), qn * id, T(0), qn * ux * id * id};
  const T duy[4] = {T(0), T(0), qn * id, qn * uy * id * id};
  const T dd[4] = {T(0), -qn * ux * id * id, -qn * uy * id * id, -qn * u2 * id * id * id};
  T l[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double v, gxv, gyv;
    interp(a.lam_dep[c], X, Y, nx, v, gxv, gyv);
    l[0] += val[c] * static_cast<T>(gxv);
    l[1] += val[c] * static_cast<T>(gyv);
    l[2] += dux[c] * static_cast<T>(v);
    l[3] += duy[c] * static_cast<T>(v);
    if (un) l[4] += dd[c] * static_cast<T>(v);
  }
#pragma unroll
  for (int c = 0; c < 5; ++c) store_at(a.lam_y + c * np, p, ly[c] + l[c]);
}

// ------------------------------------------------------------------ grid side

// out[c] = cotangent of field c at slice k (node layout, T; boundary nodes
// dropped) + extra[c] (FP64 stored layout); both may be null.  With `loss`
// set it also adds sum_c <cot[c], field[c]> to *loss (one atomic per
// workgroup of a grid held to kLossBlocks).
constexpr unsigned kLossBlocks = 1024;

template <typename T>
__global__ void __launch_bounds__(kBlock) k_adj_seed(Geom g, AdjSeedArgs<T> a) {
  const int n = g.nx * g.ny;
  const int stride = static_cast<int>(gridDim.x) * kBlock;
  double s = 0.0;
  for (int e = static_cast<int>(blockIdx.x) * kBlock + static_cast<int>(threadIdx.x); e < n; e += stride) {
    const int i = e & (g.nx - 1), j = e >> g.lx;
    const bool interior = i > 0 && j > 0;
    const int nodes = j * (g.nx + 1) + i;
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      double v = 0.0;
      if (interior && a.cot[c]) {
        v = static_cast<double>(a.cot[c][nodes]);
        if (a.loss) s += v * static_cast<double>(a.field[c][e]);
      }
      if (a.extra[c]) v += a.extra[c][e];
      a.out[c][e] = v;
    }
  }
  if (!a.loss) return;
  __shared__ double red[kBlock / 64];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0;
    for (int w = 0; w < kBlock / 64; ++w) t += red[w];
    gadd(a.loss, t);
  }
}

// Source assembly of an adjoint solve + forward transform along x, field by
// field (blockIdx.y):  s = p0 + d_x p1 + d_y p2 (FP64 planes, p1 and p2 may
// be null), and for an earlier predictor-corrector iteration, whose p0 holds
// only what the trial push scattered, s = p0 - shift lsb with the solved
// source lsb of the iteration after it; p0 is then cleared for the next
// scatter and lsb joins `sum` (stored or added), from which the slice's
// Jz and J_perp adjoints are formed once.  Zero on the Dirichlet nodes.
template <typename T, int LOGN>
__global__ void __launch_bounds__(kBlock, dst_blocks_per_cu(LOGN, sizeof(T)))
k_adj_src(Geom g, AdjSrcArgs<T> a, AxisTables<T> tx) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  const int j0 = xcd_strip(blockIdx.x, gridDim.x) * R;
  const int fld = blockIdx.y;
  const double ihx = 0.5 / g.hx, ihy = 0.5 / g.hy;
  double* __restrict__ p0 = a.p0[fld];
  const double* __restrict__ p1 = a.p1[fld];
  const double* __restrict__ p2 = a.p2[fld];
  const T* __restrict__ lsb = a.lsb[fld];
  double* __restrict__ sum = a.sum[fld];
  struct In {
    double c, e, w, n, s;
    T l;
    __device__ void pin() {
      dst_detail::pin(c);
      dst_detail::pin(e);
      dst_detail::pin(w);
      dst_detail::pin(n);
      dst_detail::pin(s);
      dst_detail::pin(l);
    }
  };
  for_row_batches<R, LOGN, src_batch<T, LOGN>(), In>(
      [&](int e, In& v) {
        const int i = e & (n - 1), j = j0 + (e >> LOGN);
        const int o = j * n + i;
        v = In{load_at<double>(p0, o), 0.0, 0.0, 0.0, 0.0, T(0)};
        if (p1) {
          v.e = load_at(p1, i + 1 < n ? o + 1 : o);
          v.w = load_at(p1, i > 0 ? o - 1 : o);
          v.n = load_at(p2, j + 1 < g.ny ? o + n : o);
          v.s = load_at(p2, j > 0 ? o - n : o);
        }
        if (lsb) {
          v.l = load_at(lsb, o);
          if (a.sum_add) v.e = load_at<double>(sum, o);   // an iteration's source has no derivative part
        }
      },
      [&](int, int e, const In& v) {
        const int r = e >> LOGN, i = e & (n - 1), j = j0 + r;
        const int o = j * n + i;
        double s = v.c;
        if (p1)
          s += ((i + 1 < n ? v.e : 0.0) - (i > 1 ? v.w : 0.0)) * ihx +
               ((j + 1 < g.ny ? v.n : 0.0) - (j > 1 ? v.s : 0.0)) * ihy;
        if (lsb) {
          const double l = static_cast<double>(v.l);
          s -= a.shift * l;
          p0[o] = 0.0;
          sum[o] = a.sum_add ? v.e + l : l;
        }
        buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)] = static_cast<T>((i > 0 && j > 0) ? s : 0.0);
      });
  xf.commit();
  __syncthreads();
  block_dst<T, LOGN, true>(buf, ppitch, xf);
  rows_to_plane<T, R, LOGN>(g, j0, buf, ppitch, a.out + static_cast<size_t>(fld) * g.nx * g.ny);
}

// End of a slice on the grid.  With S the sum over the iterations of the
// solved corrector sources lsb (the first iteration's still in lsb0, the
// others in `sum`) and the solved psi, Ez, Bz adjoint sources:
//   lam_Jz = d_y S_x - d_x S_y,   lam_R = -lpsi,
//   lam_Jx = carry_jx - d_x lez - d_y lbz,  lam_Jy = carry_jy - d_y lez + d_x lbz,
//   carry to slice k-1: J_perp (-S_y, S_x) / 2dz;
//   initial guess B^0 = 2 B_{k-1} - B_{k-2} transposed: with
//   L0 = lam_b - shift lsb0,  b1 = b2 + 2 L0 (with what slice k+1 handed to
//   B_{k-1}) and b2 = -L0;  lam_b cleared for the next slice's scatter;
//   dL/da_k = -<lam_Jz, G>, dL/dsigma = -a_k <lam_Jz, dG/dsigma> as partial
//   records.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_adj_dep_grid(Geom g, AdjDepGridArgs<T> a) {
  const int nx = g.nx, ny = g.ny;
  const int n = nx * ny;
  const double ihx = 0.5 / g.hx, ihy = 0.5 / g.hy;
  double acc[3] = {0.0, 0.0, 0.0};
  const int stride = static_cast<int>(gridDim.x) * kBlock;
  for (int e = static_cast<int>(blockIdx.x) * kBlock + static_cast<int>(threadIdx.x); e < n; e += stride) {
    const int i = e & (nx - 1), j = e >> g.lx;
    const bool in = i > 0 && j > 0;
    // neighbours with clamped indices; values on the Dirichlet nodes are zero
    const int oe = i + 1 < nx ? e + 1 : e, ow = i > 0 ? e - 1 : e;
    const int on = j + 1 < ny ? e + nx : e, os = j > 0 ? e - nx : e;
    const bool he = i + 1 < nx, hw = i > 1, hn = j + 1 < ny, hs = j > 1;
    auto val = [&](const T* l, const double* s, int o) {
      const double v = static_cast<double>(l[o]);
      return s ? v + s[o] : v;
    };
    const double l0x = static_cast<double>(a.lsb_x[e]), l0y = static_cast<double>(a.lsb_y[e]);
    const double sx = a.sum_x ? l0x + a.sum_x[e] : l0x, sy = a.sum_y ? l0y + a.sum_y[e] : l0y;
    const double sx_n = val(a.lsb_x, a.sum_x, on), sx_s = val(a.lsb_x, a.sum_x, os);
    const double sy_e = val(a.lsb_y, a.sum_y, oe), sy_w = val(a.lsb_y, a.sum_y, ow);
    const double ez_e = a.lez[oe], ez_w = a.lez[ow], ez_n = a.lez[on], ez_s = a.lez[os];
    const double bz_e = a.lbz[oe], bz_w = a.lbz[ow], bz_n = a.lbz[on], bz_s = a.lbz[os];
    const double r = a.lpsi[e];
    const double cjx = a.carry_jx[e], cjy = a.carry_jy[e];
    const double l0bx = a.lam_bx[e] - a.shift * l0x, l0by = a.lam_by[e] - a.shift * l0y;
    const double b2x = a.b2x[e], b2y = a.b2y[e];
    auto diff = [](double p, bool hp, double m, bool hm) { return (hp ? p : 0.0) - (hm ? m : 0.0); };
    const double lz = diff(sx_n, hn, sx_s, hs) * ihy - diff(sy_e, he, sy_w, hw) * ihx;
    const double jx = cjx - diff(ez_e, he, ez_w, hw) * ihx - diff(bz_n, hn, bz_s, hs) * ihy;
    const double jy = cjy - diff(ez_n, hn, ez_s, hs) * ihy + diff(bz_e, he, bz_w, hw) * ihx;
    if (in) {
      acc[0] += lz * a.bgx[i] * a.bgy[j];
      acc[1] += lz * a.dbgx[i] * a.bgy[j];
      acc[2] += lz * a.bgx[i] * a.dbgy[j];
    }
    a.lam_r[e] = in ? -r : 0.0;
    a.lam_jx[e] = in ? jx : 0.0;
    a.lam_jy[e] = in ? jy : 0.0;
    a.lam_jz[e] = in ? lz : 0.0;
    a.jp_x[e] = -sy * a.inv2dz;
    a.jp_y[e] = sx * a.inv2dz;
    a.b1x[e] = b2x + 2.0 * l0bx;
    a.b1y[e] = b2y + 2.0 * l0by;
    a.b2x[e] = -l0bx;
    a.b2y[e] = -l0by;
    a.lam_bx[e] = 0.0;
    a.lam_by[e] = 0.0;
  }
  partials::store<3>(acc, a.part, static_cast<int>(blockIdx.x));
}

template <typename T>
__global__ void k_copy_particles(Lattice L, Particles<T> src, Particles<T> dst, int k, T dz) {
  const size_t np = static_cast<size_t>(L.np);
  const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
  // history slots of f_{k-1}, ..., f_{k-4}
  const int s1 = (k + 3) & 3, s2 = (k + 2) & 3, s3 = (k + 1) & 3, s4 = k & 3;
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < np; i += stride) {
    T y[5] = {src.xi_x[i], src.xi_y[i], src.ux[i], src.uy[i], src.psi[i]};
    dst.xi_x[i] = y[0];
    dst.xi_y[i] = y[1];
    dst.ux[i] = y[2];
    dst.uy[i] = y[3];
    dst.psi[i] = y[4];
    dst.w[i] = src.w[i];
#pragma unroll
    for (int c = 0; c < 20; ++c) dst.hist[c * np + i] = src.hist[c * np + i];
    if (dst.pab) {
      const T* h = src.hist;
#pragma unroll
      for (int c = 0; c < 5; ++c)
        dst.pab[c * np + i] = ab5_history(y[c], h[(s1 * 5 + c) * np + i], h[(s2 * 5 + c) * np + i],
                                          h[(s3 * 5 + c) * np + i], h[(s4 * 5 + c) * np + i], dz);
    }
  }
}

template <typename T, typename U>
__global__ void k_copy_planes(size_t n, int count, CopyPlanes<T, U> c) {
  const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
  for (size_t e = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; e < n; e += stride)
    for (int q = 0; q < count; ++q) c.dst[q][e] = static_cast<U>(c.src[q][e]);
}

// ------------------------------------------------------------------ launchers
namespace {
dim3 g1(size_t n) {
  size_t b = (n + kBlock - 1) / kBlock;
  if (b > 8192) b = 8192;
  if (b == 0) b = 1;
  return dim3(static_cast<unsigned>(b));
}
dim3 gp(int64_t n) {
  int64_t b = (n + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  return dim3(static_cast<unsigned>(b));
}

// the adjoint needs a shape with a derivative: orders 1-3
template <typename F>
void with_adj_order(int order, F&& f) {
  switch (order) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    default: throw std::invalid_argument("the adjoint needs a shape order of 1, 2 or 3");
  }
}
}  // namespace

template <typename T>
void launch_adj_push(const Geom& g, const Lattice& L, const AdjPushArgs<T>& a, bool trial,
                     hipStream_t st) {
  const push_detail::TileShape ts = push_detail::tile_shape(L, a.tile_rows, a.tile_halo);
  const size_t lds = static_cast<size_t>(6) * ts.nw * ts.nh * sizeof(double);
  if (lds > 160 * 1024) throw std::invalid_argument("adjoint push histogram exceeds the LDS");
  const dim3 grid(L.nX / ts.tx, L.nY / ts.ty);
  with_adj_order(g.order, [&](auto order) {
    constexpr int O = decltype(order)::value;
    const void* fn = trial ? reinterpret_cast<const void*>(&k_adj_push<T, 1, O>)
                           : reinterpret_cast<const void*>(&k_adj_push<T, 0, O>);
    if (lds > 65536)
      QSP_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    if (trial)
      hipLaunchKernelGGL((k_adj_push<T, 1, O>), grid, dim3(kBlock), lds, st, g, L, a);
    else
      hipLaunchKernelGGL((k_adj_push<T, 0, O>), grid, dim3(kBlock), lds, st, g, L, a);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_adj_trial_later(const Geom& g, const Lattice& L, const AdjPushArgs<T>& a,
                            hipStream_t st) {
  if (!a.rec || !a.acc || (a.acc_mode != 1 && a.acc_mode != 2))
    throw std::invalid_argument("a later trial push transpose needs the record and the sums");
  const push_detail::TileShape ts = push_detail::tile_shape(L, a.tile_rows, a.tile_halo);
  const size_t lds = static_cast<size_t>(2) * ts.nw * ts.nh * sizeof(double);
  if (lds > 160 * 1024) throw std::invalid_argument("adjoint push histogram exceeds the LDS");
  const dim3 grid(L.nX / ts.tx, L.nY / ts.ty);
  with_adj_order(g.order, [&](auto order) {
    constexpr int O = decltype(order)::value;
    if (lds > 65536)
      QSP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_adj_trial_later<T, O>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    hipLaunchKernelGGL((k_adj_trial_later<T, O>), grid, dim3(kBlock), lds, st, g, L, a);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_adj_deposit(const Geom& g, const Lattice& L, const AdjDepArgs<T>& a, hipStream_t st) {
  with_adj_order(g.order, [&](auto order) {
    hipLaunchKernelGGL((k_adj_deposit<T, decltype(order)::value>), gp(L.np), dim3(kBlock), 0, st,
                       g, L, a);
  });
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_adj_seed(const Geom& g, const AdjSeedArgs<T>& a, hipStream_t st) {
  dim3 grid = g1(static_cast<size_t>(g.nx) * g.ny);
  if (a.loss && grid.x > kLossBlocks) grid.x = kLossBlocks;
  hipLaunchKernelGGL(k_adj_seed<T>, grid, dim3(kBlock), 0, st, g, a);
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_adj_src(const Geom& g, const AdjSrcArgs<T>& a, const AxisTables<T>& tx, hipStream_t st) {
  if (a.count < 1 || a.count > 3) throw std::invalid_argument("adjoint source: 1..3 planes");
  for (int q = 0; q < a.count; ++q)
    if (!a.p0[q] || (a.p1[q] != nullptr) != (a.p2[q] != nullptr) || (a.lsb[q] && (!a.sum[q] || a.p1[q])))
      throw std::invalid_argument("adjoint source: missing planes");
  const int R = pass_rows<T>(g.nx);
  const size_t lds = pass_lds<T>(R, g.nx);
  with_logn(g.nx, [&](auto e) {
    constexpr int E = decltype(e)::value;
    if (lds > 65536)
      QSP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_adj_src<T, E>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    hipLaunchKernelGGL((k_adj_src<T, E>), dim3(g.ny / R, a.count), dim3(kBlock), lds, st, g, a, tx);
  });
  QSP_LAUNCH_CHECK();
}

int adj_part_count(const Geom& g) {
  const int b = (g.nx * g.ny + kBlock - 1) / kBlock;
  return b < 2048 ? b : 2048;
}

template <typename T>
void launch_adj_dep_grid(const Geom& g, const AdjDepGridArgs<T>& a, hipStream_t st) {
  hipLaunchKernelGGL(k_adj_dep_grid<T>, dim3(adj_part_count(g)), dim3(kBlock), 0, st, g, a);
  QSP_LAUNCH_CHECK();
}

template <typename T>
void launch_copy_particles(const Lattice& L, const Particles<T>& src, const Particles<T>& dst,
                           int k, double dzeta, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_particles<T>, g1(static_cast<size_t>(L.np)), dim3(kBlock), 0, st, L, src,
                     dst, k, static_cast<T>(dzeta));
  QSP_LAUNCH_CHECK();
}

template <typename T, typename U>
void launch_copy_planes(size_t n, int count, const CopyPlanes<T, U>& c, hipStream_t st) {
  if (count == 0) return;
  hipLaunchKernelGGL((k_copy_planes<T, U>), g1(n), dim3(kBlock), 0, st, n, count, c);
  QSP_LAUNCH_CHECK();
}

#define QSP_INST(T)                                                                             \
  template void launch_adj_push<T>(const Geom&, const Lattice&, const AdjPushArgs<T>&, bool,    \
                                   hipStream_t);                                               \
  template void launch_adj_trial_later<T>(const Geom&, const Lattice&, const AdjPushArgs<T>&,   \
                                          hipStream_t);                                        \
  template void launch_adj_deposit<T>(const Geom&, const Lattice&, const AdjDepArgs<T>&,        \
                                      hipStream_t);                                            \
  template void launch_adj_seed<T>(const Geom&, const AdjSeedArgs<T>&, hipStream_t);            \
  template void launch_adj_dep_grid<T>(const Geom&, const AdjDepGridArgs<T>&, hipStream_t);     \
  template void launch_adj_src<T>(const Geom&, const AdjSrcArgs<T>&, const AxisTables<T>&,      \
                                  hipStream_t);                                                \
  template void launch_copy_particles<T>(const Lattice&, const Particles<T>&,                   \
                                         const Particles<T>&, int, double, hipStream_t);        \
  template void launch_copy_planes<T, T>(size_t, int, const CopyPlanes<T, T>&, hipStream_t);
QSP_INST(float)
QSP_INST(double)
#undef QSP_INST

}  // namespace qsp
