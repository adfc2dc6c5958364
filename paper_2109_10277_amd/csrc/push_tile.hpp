// Device-side body of the fused plasma gather + Adams-Bashforth push +
// deposit (HiPACE++, arXiv:2109.10277, Sec. III.B: plasma pusher equations;
// deposition zeroth order in zeta, transverse shape of order 0-3).
//
// Particles are stored SoA in lattice order and keep their lattice site for
// life; positions are stored as displacements from that site (in cells) so
// that small displacements keep full precision.  A workgroup owns a tile of
// lattice sites; its particles deposit into FP64 histograms in LDS covering
// the tile's cells plus a halo, which are then added to the global FP64
// deposit arrays: the nodes of the tile's own cells with plain stores, the
// halo nodes with one atomic per non-zero node into shared planes (DepOut).
// Particles that have left the tile+halo fall back to global FP64 atomics.
#pragma once

#include "common.hpp"
#include "kernels.hpp"
#include "shape.hpp"

namespace qsp {
namespace push_detail {

struct TileShape {
  int tx, ty;      // lattice sites per tile (tx a power of two)
  int ltx;         // log2 tx
  int lpx, lpy;    // log2 ppc
  int nw, nh;      // LDS node tile (cells + 1 + 2 halo)
  int halo;        // cells around the tile's own cells covered in LDS
};

__host__ __device__ inline int ilog2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

__host__ __device__ inline TileShape tile_shape(const Lattice& L, int rows, int halo) {
  TileShape t;
  t.halo = halo;
  t.tx = L.nX < 64 ? L.nX : 64;
  t.ty = L.nY < rows ? L.nY : rows;
  t.ltx = ilog2(t.tx);
  t.lpx = ilog2(L.ppc_x);
  t.lpy = ilog2(L.ppc_y);
  t.nw = (t.tx >> t.lpx) + 1 + 2 * halo;
  t.nh = (t.ty >> t.lpy) + 1 + 2 * halo;
  return t;
}

// Tile column of the workgroup, its row being blockIdx.y.  Workgroups go round-
// robin to the 8 XCDs, so with whole rows of tiles a column of tiles would stay
// on one XCD, and the expensive tiles, those of the wake around the axis (same-
// address LDS atomics, particles outside their tile), on two or three of them:
// each row starts one tile further on.  1024^2 with 2x2 particles: real push
// 224 -> 186 us, later trial 79 -> 67, first trial 116 -> 99; one particle a
// cell: real push 69.9 -> 65.7.  The price is the field rows that vertical
// neighbours no longer share in an L2: with 16 tiles a row or fewer it takes
// what the trial pushes gain (1024^2: 20.3 against 19.6 us in quiet plasma, no
// difference in the wake; 512^2 box 23.46 against 23.36 ms), so these rotate
// from 32 tiles a row up.
__device__ __forceinline__ int tile_column(bool real_push) {
  const unsigned int gx = gridDim.x;   // a power of two, like the lattice
  return static_cast<int>(real_push || gx >= 32 ? (blockIdx.x + blockIdx.y) & (gx - 1) : blockIdx.x);
}

// Index of particle e of the tile at site (I0, J0) (the tile's first one for e
// beyond it).
__device__ __forceinline__ unsigned int tile_particle(const Lattice& L, const TileShape& ts, int I0,
                                                      int J0, int e) {
  const int ec = e < ts.tx * ts.ty ? e : 0;
  return static_cast<unsigned int>(J0 + (ec >> ts.ltx)) * static_cast<unsigned int>(L.nX) +
         static_cast<unsigned int>(I0 + (ec & (ts.tx - 1)));
}

template <typename T>
__device__ inline bool inside(int c0, T t, int n) {
  const T fl = floor(t);
  const int c = c0 + static_cast<int>(fl);
  return c >= 0 && (c < n || (c == n && t == fl));
}

// Keeps a loaded value where it was loaded: without it the compiler moves a
// load next to its first use, behind the particle's decisions, and a batch of
// loads becomes a chain of memory round trips.
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

// CIC interpolation in cell (i, j), 0 <= i < nx, 0 <= j < ny, of several
// planes; the upper Dirichlet nodes (index n, not stored) are zero.  The two
// nodes of a row come with one load of two values (aligned to one value
// only), clamped to stay in the row: half the load instructions and
// addresses of a load per node.  32-bit offsets (a plane is below 4 GiB).
template <typename T>
struct Cic {
  T w00, w10, w01, w11;
  unsigned int r0, r1;   // offsets of the pairs of rows j, j + 1
  bool ie, jn;           // node i + 1 (j + 1) is stored
  struct alignas(sizeof(T)) Two {
    T a, b;
  };
  struct Node {          // the four nodes of a plane
    T a0, b0, a1, b1;
    __device__ __forceinline__ void pin() {
      push_detail::pin(a0);
      push_detail::pin(b0);
      push_detail::pin(a1);
      push_detail::pin(b1);
    }
  };
  __device__ __forceinline__ void at(int i, int j, T fx, T fy, int nx, int ny) {
    w00 = (T(1) - fx) * (T(1) - fy);
    w10 = fx * (T(1) - fy);
    w01 = (T(1) - fx) * fy;
    w11 = fx * fy;
    ie = i + 1 < nx;
    jn = j + 1 < ny;
    const int i0 = ie ? i : i - 1;   // nx >= 16
    r0 = static_cast<unsigned int>(j * nx + i0);
    r1 = jn ? r0 + static_cast<unsigned int>(nx) : r0;
  }
  __device__ __forceinline__ Node load(const T* __restrict__ F) const {
    const char* f = reinterpret_cast<const char*>(F);
    const Two u = *reinterpret_cast<const Two*>(f + r0 * static_cast<unsigned int>(sizeof(T)));
    const Two v = *reinterpret_cast<const Two*>(f + r1 * static_cast<unsigned int>(sizeof(T)));
    return {u.a, u.b, v.a, v.b};
  }
  __device__ __forceinline__ T sum(const Node& f) const {
    const T f00 = ie ? f.a0 : f.b0, f01 = ie ? f.a1 : f.b1;
    return w00 * f00 + w10 * (ie ? f.b0 : T(0)) + w01 * (jn ? f01 : T(0)) +
           w11 * ((ie && jn) ? f.b1 : T(0));
  }
};

__device__ inline void lds_add(double* p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ inline void global_add(double* p, double v) { unsafeAtomicAdd(p, v); }

// Adds the nch channels of a tile histogram (nw x nh nodes starting at
// global node (ox, oy), channel c at tile + c * nw * nh) to the global FP64
// planes ch[c]: one atomic per stored, non-zero node.  Nodes are walked in
// row-major order, kBlock at a time, with a running (row, column) pair
// instead of divisions, and the channel loop is unrolled so that each
// plane's address is a compile-time argument offset: no load, and so no
// wait on the atomics already in flight, precedes an atomic.
template <int nch>
__device__ __forceinline__ void flush_tile(double* const* ch, const double* tile,
                                           const TileShape& ts, int ox, int oy, int nx, int ny) {
  const int ntile = ts.nw * ts.nh;
  const int step_r = kBlock / ts.nw, step_c = kBlock % ts.nw;
  int r = threadIdx.x / ts.nw, cl = threadIdx.x % ts.nw;
  for (int l = threadIdx.x; l < ntile; l += kBlock) {
    const int gi = ox + cl, gj = oy + r;
    if (gi >= 1 && gi < nx && gj >= 1 && gj < ny) {
      const size_t o = static_cast<size_t>(gj) * nx + gi;
      double val[nch];
#pragma unroll
      for (int c = 0; c < nch; ++c) val[c] = tile[c * ntile + l];
#pragma unroll
      for (int c = 0; c < nch; ++c)
        if (val[c] != 0.0) global_add(ch[c] + o, val[c]);
    }
    r += step_r;
    cl += step_c;
    if (cl >= ts.nw) {
      cl -= ts.nw;
      ++r;
    }
  }
}

// Owner form of flush_tile: the nodes of the tile's own cells (local
// columns halo .. halo + tx/ppc_x - 1, rows likewise) are stored into ch[c],
// zeros included; the other non-zero nodes are added to sh[c] with atomics.
template <int nch>
__device__ __forceinline__ void flush_tile_owned(double* const* ch, double* const* sh,
                                                 const double* tile, const TileShape& ts, int ox,
                                                 int oy, int nx, int ny) {
  const int ntile = ts.nw * ts.nh;
  const unsigned int ocx = static_cast<unsigned int>(ts.tx >> ts.lpx);
  const unsigned int ocy = static_cast<unsigned int>(ts.ty >> ts.lpy);
  const int step_r = kBlock / ts.nw, step_c = kBlock % ts.nw;
  int r = threadIdx.x / ts.nw, cl = threadIdx.x % ts.nw;
  for (int l = threadIdx.x; l < ntile; l += kBlock) {
    const int gi = ox + cl, gj = oy + r;
    if (gi >= 1 && gi < nx && gj >= 1 && gj < ny) {
      const size_t o = static_cast<size_t>(gj) * nx + gi;
      const bool own = static_cast<unsigned int>(cl - ts.halo) < ocx &&
                       static_cast<unsigned int>(r - ts.halo) < ocy;
      double val[nch];
#pragma unroll
      for (int c = 0; c < nch; ++c) val[c] = tile[c * ntile + l];
#pragma unroll
      for (int c = 0; c < nch; ++c) {
        if (own)
          ch[c][o] = val[c];
        else if (val[c] != 0.0)
          global_add(sh[c] + o, val[c]);
      }
    }
    r += step_r;
    cl += step_c;
    if (cl >= ts.nw) {
      cl -= ts.nw;
      ++r;
    }
  }
}

__device__ inline unsigned long long block_sum(unsigned int v, unsigned int* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  unsigned long long s = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kBlock / 64; ++w) s += red[w];
  return s;
}

// Deposit of one particle: nch values v at offset (xi, eta) from its
// lattice cell origin (ci0 + fx0, cj0 + fy0) into the tile histogram, or
// straight to the global planes (the shared ones for an owner flush) when
// the stencil leaves the tile (counted in nglob).  A particle that is not
// live deposits zeros into the histogram and nothing outside it.
template <typename T, int O, int nch>
__device__ __forceinline__ void deposit_particle(const DepOut& dep, double* tile, const TileShape& ts,
                                                 int ox, int oy, int nx, int ny, bool tiled,
                                                 bool owner, int ci0,
                                                 int cj0, T fx0, T fy0, T xi, T eta,
                                                 const double (&v)[4], unsigned int& nglob,
                                                 bool live = true) {
  const int ntile = ts.nw * ts.nh;
  int bi, bj;
  const T dx = shape::locate<O>(ci0, fx0 + xi, nx, bi);
  const T dy = shape::locate<O>(cj0, fy0 + eta, ny, bj);
  double sx[O + 1], sy[O + 1];
  shape::weights<O>(static_cast<double>(dx), sx);
  shape::weights<O>(static_cast<double>(dy), sy);
  const int li = bi - ox, lj = bj - oy;
  if (tiled && li >= 0 && li + O < ts.nw && lj >= 0 && lj + O < ts.nh) {
    const int base = lj * ts.nw + li;
#pragma unroll
    for (int c = 0; c < nch; ++c) {
      double* t = tile + c * ntile + base;
#pragma unroll
      for (int qb = 0; qb <= O; ++qb)
#pragma unroll
        for (int qa = 0; qa <= O; ++qa) lds_add(t + qb * ts.nw + qa, v[c] * (sx[qa] * sy[qb]));
    }
  } else if (live) {
    if (tiled) ++nglob;
#pragma unroll
    for (int qb = 0; qb <= O; ++qb) {
      const int gj = bj + qb;
#pragma unroll
      for (int qa = 0; qa <= O; ++qa) {
        const int gi = bi + qa;
        if (gi < 1 || gi >= nx || gj < 1 || gj >= ny) continue;
        const size_t o = static_cast<size_t>(gj) * nx + gi;
        const double s = sx[qa] * sy[qb];
#pragma unroll
        for (int c = 0; c < nch; ++c) global_add((owner ? dep.sh[c] : dep.ch[c]) + o, v[c] * s);
      }
    }
  }
}

// Bx, By at displacement (xk, ek) from the lattice cell origin
// (ci0 + fx0, cj0 + fy0), shape order O (indices clamped: always in bounds).
template <typename T, int O>
__device__ __forceinline__ void gather_bxby(const SliceFields<T>& f, int ci0, int cj0, T fx0, T fy0,
                                            T xk, T ek, int nx, int ny, T& bx, T& by) {
  if constexpr (O == 1) {
    int ci, cj;
    const T fx = shape::locate<1>(ci0, fx0 + xk, nx, ci);
    const T fy = shape::locate<1>(cj0, fy0 + ek, ny, cj);
    Cic<T> cic;
    cic.at(ci, cj, fx, fy, nx, ny);
    const auto nb = cic.load(f.bx), mb = cic.load(f.by);
    bx = cic.sum(nb);
    by = cic.sum(mb);
  } else {
    int bi, bj;
    const T dx = shape::locate<O>(ci0, fx0 + xk, nx, bi);
    const T dy = shape::locate<O>(cj0, fy0 + ek, ny, bj);
    T wx[O + 1], wy[O + 1];
    int ix[O + 1], iy[O + 1];
    bool okx[O + 1], oky[O + 1];
    shape::weights<O>(dx, wx);
    shape::weights<O>(dy, wy);
    shape::axis_nodes<O>(bi, nx, ix, okx);
    shape::axis_nodes<O>(bj, ny, iy, oky);
#pragma unroll
    for (int q = 0; q <= O; ++q) {
      wx[q] = okx[q] ? wx[q] : T(0);
      wy[q] = oky[q] ? wy[q] : T(0);
    }
    bx = shape::interp<O>(f.bx, ix, iy, wx, wy, nx);
    by = shape::interp<O>(f.by, ix, iy, wx, wy, nx);
  }
}

// Trial push of a later predictor-corrector iteration for the particles of
// the tile at lattice site (I0, J0).  Between iterations only Bx, By
// change, and they enter the push as a kick -dz b0 (By, -Bx) on the
// momentum: the new position, Psi and the rest of the momentum come from the
// slice's first trial push (the record), and Bx, By are gathered at the
// slice-k position as there.  A thread takes kLaterBatch particles at a
// time (FP32 linear shape; one otherwise, whose registers two would crowd)
// and issues all their loads, then all their gathers, before its first
// deposit; a particle without deposit (record factor 0) adds zeros, so that
// nothing waits on the factor.
constexpr int kLaterBatch = 2;

template <typename T, int O, int nch>
struct LaterBatch {
  static constexpr int U = sizeof(T) == 4 && O == 1 ? kLaterBatch : 1;
  T fac[U], xk[U], ek[U], xn[U], en[U], cx[U], cy[U];

  static __device__ __forceinline__ void site(const TileShape& ts, int I0, int J0, int e, int& I, int& J) {
    const int ec = e < ts.tx * ts.ty ? e : 0;   // a missing particle reads the tile's first
    I = I0 + (ec & (ts.tx - 1));
    J = J0 + (ec >> ts.ltx);
  }
  __device__ __forceinline__ void load(const Lattice& L, const PushArgs<T>& a, const TileShape& ts,
                                       int I0, int J0, int e0) {
    const size_t np = static_cast<size_t>(L.np);
    const T* r = a.rec;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int I, J;
      site(ts, I0, J0, e0 + u * kBlock + static_cast<int>(threadIdx.x), I, J);
      // 32-bit offsets from uniform plane bases (the launch checks that a
      // particle plane is below 4 GiB)
      const unsigned int p = static_cast<unsigned int>(J) * static_cast<unsigned int>(L.nX) +
                             static_cast<unsigned int>(I);
      xk[u] = load_at(a.p.xi_x, p);
      ek[u] = load_at(a.p.xi_y, p);
      const T* q = r;
      xn[u] = load_at(q, p);
      en[u] = load_at(q += np, p);
      cx[u] = load_at(q += np, p);
      cy[u] = load_at(q += np, p);
      fac[u] = load_at(q += np, p);
    }
    // keep the scheduler from moving a later particle's loads behind an
    // earlier one's gather (the wait for a load also waits for every load
    // issued before it)
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void deposit(const Lattice& L, const PushArgs<T>& a, double* tile,
                                          const TileShape& ts, int I0, int J0, int e0, int ox, int oy,
                                          int nx, int ny, bool tiled, bool owner, unsigned int& nglob) {
    const T kick = static_cast<T>(a.dzeta) * T(kAB5[0]);
    T bx[U], by[U], fx0[U], fy0[U];
    int ci0[U], cj0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int I, J;
      site(ts, I0, J0, e0 + u * kBlock + static_cast<int>(threadIdx.x), I, J);
      ci0[u] = I >> ts.lpx;
      cj0[u] = J >> ts.lpy;
      fx0[u] = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
      fy0[u] = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
      pin(xk[u]);
      pin(ek[u]);
    }
    if constexpr (O == 1) {
      // the gather of every particle of the batch: addresses and weights,
      // then all loads, then the sums
      Cic<T> cic[U];
      typename Cic<T>::Node gx[U], gy[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int ci, cj;
        const T fx = shape::locate<1>(ci0[u], fx0[u] + xk[u], nx, ci);
        const T fy = shape::locate<1>(cj0[u], fy0[u] + ek[u], ny, cj);
        cic[u].at(ci, cj, fx, fy, nx, ny);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        gx[u] = cic[u].load(a.f.bx);
        gy[u] = cic[u].load(a.f.by);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        gx[u].pin();
        gy[u].pin();
        bx[u] = cic[u].sum(gx[u]);
        by[u] = cic[u].sum(gy[u]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
        gather_bxby<T, O>(a.f, ci0[u], cj0[u], fx0[u], fy0[u], xk[u], ek[u], nx, ny, bx[u],
                          by[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (e0 + u * kBlock + static_cast<int>(threadIdx.x) >= ts.tx * ts.ty) continue;
      const bool live = fac[u] != T(0);   // selects, not branches
      const double v[4] = {live ? static_cast<double>(fac[u] * (cx[u] - kick * by[u])) : 0.0,
                           live ? static_cast<double>(fac[u] * (cy[u] + kick * bx[u])) : 0.0, 0.0,
                           0.0};
      deposit_particle<T, O, nch>(a.dep, tile, ts, ox, oy, nx, ny, tiled, owner, ci0[u], cj0[u],
                                  fx0[u], fy0[u], xn[u], en[u], v, nglob, live);
    }
  }
};

// What a particle's push reads of the particle itself, all issued at once: the
// state, the history part P_k of the step (left by the previous real push)
// and, for the real push, f_{k-1}, f_{k-2}, f_{k-3}, which form P_{k+1} with
// f_k.  A thread beyond the tile reads the tile's first particle.  The pushes
// are bound by bytes and atomics, so the round trips saved show little: 1024^2
// FP32 real push 71.0 -> 69.9 us, first trial 35.9 -> 34.3.
template <typename T, int MODE>
struct ParticleLoad {
  T y[5], w, pk[5], h[3][5];
  __device__ __forceinline__ void load(const Lattice& L, const PushArgs<T>& a, const TileShape& ts,
                                       int I0, int J0, int e) {
    const size_t np = static_cast<size_t>(L.np);
    const unsigned int p = tile_particle(L, ts, I0, J0, e);
    y[0] = load_at(a.p.xi_x, p);
    y[1] = load_at(a.p.xi_y, p);
    y[2] = load_at(a.p.ux, p);
    y[3] = load_at(a.p.uy, p);
    y[4] = load_at(a.p.psi, p);
    w = load_at(a.p.w, p);
    if constexpr (MODE == kPushReal || MODE == kPushTrial) {
      const T* q = a.p.pab;   // planes by stepping: a product per plane is a chain of scalar work
#pragma unroll
      for (int c = 0; c < 5; ++c, q += np) pk[c] = load_at(q, p);
    }
    if constexpr (MODE == kPushReal) {
      const size_t np5 = 5 * np;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const T* q = a.p.hist + ((a.k + 3 - m) & 3) * np5;
#pragma unroll
        for (int c = 0; c < 5; ++c, q += np) h[m][c] = load_at(q, p);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

// Gather, push and deposit of the particles of lattice tile (tbx, tby) by
// one workgroup with the transverse shape of order O; `tile` is the
// workgroup's LDS histogram (nch channels of tile_shape's nw x nh nodes).
// Safe to call repeatedly from one workgroup.  The linear shape keeps a
// gather of its own (four weights, value selects at the upper edge), which
// the compiler allocates in fewer registers than the generic stencil.
template <typename T, int MODE, int O, bool TAPE = false>
__device__ __forceinline__ void push_tile(const Geom& g, const Lattice& L, const PushArgs<T>& a,
                                          DevCounters* ctr, int tbx, int tby, double* tile) {
  // channels: trial push Jx, Jy; otherwise rho - Jz, Jx, Jy, Jz
  constexpr bool trial = MODE == kPushTrial || MODE == kTrialLater;
  constexpr int nch = trial ? 2 : 4;
  __shared__ unsigned int red[kBlock / 64];
  const TileShape ts = tile_shape(L, a.tile_rows, a.tile_halo);
  const int ntile = ts.nw * ts.nh;
  const bool tiled = a.tiled != 0;
  const bool owner = tiled && a.dep.sh[0] != nullptr;
  const int I0 = tbx * ts.tx, J0 = tby * ts.ty;
  const int ox = (I0 >> ts.lpx) - ts.halo, oy = (J0 >> ts.lpy) - ts.halo;
  const int nx = g.nx, ny = g.ny;
  const T inv_hx = static_cast<T>(1.0 / a.hx), inv_hy = static_cast<T>(1.0 / a.hy);
  const T floor_d = static_cast<T>(a.psi_floor);
  const T dz = static_cast<T>(a.dzeta);
  const T b0 = T(kAB5[0]);
  const size_t np = static_cast<size_t>(L.np);
  unsigned int nclamp = 0, nabs = 0, nglob = 0;
  const int ntot = ts.tx * ts.ty;

  // The first loads are in flight while the histogram is cleared.
  ParticleLoad<T, MODE> in;
  LaterBatch<T, O, nch> later;
  if constexpr (MODE == kTrialLater)
    later.load(L, a, ts, I0, J0, 0);
  else
    in.load(L, a, ts, I0, J0, static_cast<int>(threadIdx.x));
  if (tiled) {
    __syncthreads();   // a previous tile's flush has read the histogram
    for (int e = threadIdx.x; e < nch * ntile; e += kBlock) tile[e] = 0.0;
    __syncthreads();
  }
  if constexpr (MODE == kTrialLater) {
    constexpr int step = LaterBatch<T, O, nch>::U * kBlock;
    for (int e0 = 0;;) {
      later.deposit(L, a, tile, ts, I0, J0, e0, ox, oy, nx, ny, tiled, owner, nglob);
      e0 += step;
      if (e0 >= ntot) break;
      later.load(L, a, ts, I0, J0, e0);
    }
  }
  for (int e = threadIdx.x; MODE != kTrialLater && e < ntot; e += kBlock) {
    if (e >= kBlock) in.load(L, a, ts, I0, J0, e);
    const int I = I0 + (e & (ts.tx - 1)), J = J0 + (e >> ts.ltx);
    const unsigned int p = static_cast<unsigned int>(J) * static_cast<unsigned int>(L.nX) +
                           static_cast<unsigned int>(I);
    T xi = in.y[0], eta = in.y[1], ux = in.y[2], uy = in.y[3], psi = in.y[4];
    const T w = in.w;
    pin(xi);
    pin(eta);
    const int ci0 = I >> ts.lpx, cj0 = J >> ts.lpy;
    const T fx0 = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
    const T fy0 = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
    bool alive = w != T(0);

    if (MODE != kDepositOnly) {
      if constexpr (MODE == kPushTrial && TAPE) {
        // the state the reverse pass of this slice starts from
        T* t = a.tape;
        store_at(t, p, xi);
        store_at(t + np, p, eta);
        store_at(t + 2 * np, p, ux);
        store_at(t + 3 * np, p, uy);
        store_at(t + 4 * np, p, psi);
        store_at(t + 5 * np, p, w);
      }
      T e1, e2, ez, bx, by, bz;
      if constexpr (O == 1) {
        int ci, cj;
        const T fx = shape::locate<1>(ci0, fx0 + xi, nx, ci);
        const T fy = shape::locate<1>(cj0, fy0 + eta, ny, cj);
        Cic<T> cic;
        cic.at(ci, cj, fx, fy, nx, ny);
        const T* const planes[6] = {a.f.exmby, a.f.eypbx, a.f.ez, a.f.bx, a.f.by, a.f.bz};
        typename Cic<T>::Node nd[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) nd[q] = cic.load(planes[q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 6; ++q) nd[q].pin();
        e1 = cic.sum(nd[0]);
        e2 = cic.sum(nd[1]);
        ez = cic.sum(nd[2]);
        bx = cic.sum(nd[3]);
        by = cic.sum(nd[4]);
        bz = cic.sum(nd[5]);
      } else {
        int bi, bj;
        const T dx = shape::locate<O>(ci0, fx0 + xi, nx, bi);
        const T dy = shape::locate<O>(cj0, fy0 + eta, ny, bj);
        T wx[O + 1], wy[O + 1];
        int ix[O + 1], iy[O + 1];
        bool okx[O + 1], oky[O + 1];
        shape::weights<O>(dx, wx);
        shape::weights<O>(dy, wy);
        shape::axis_nodes<O>(bi, nx, ix, okx);
        shape::axis_nodes<O>(bj, ny, iy, oky);
#pragma unroll
        for (int q = 0; q <= O; ++q) {
          wx[q] = okx[q] ? wx[q] : T(0);
          wy[q] = oky[q] ? wy[q] : T(0);
        }
        e1 = shape::interp<O>(a.f.exmby, ix, iy, wx, wy, nx);
        e2 = shape::interp<O>(a.f.eypbx, ix, iy, wx, wy, nx);
        ez = shape::interp<O>(a.f.ez, ix, iy, wx, wy, nx);
        bx = shape::interp<O>(a.f.bx, ix, iy, wx, wy, nx);
        by = shape::interp<O>(a.f.by, ix, iy, wx, wy, nx);
        bz = shape::interp<O>(a.f.bz, ix, iy, wx, wy, nx);
      }
      // right-hand side of the pusher equations for an electron (q = -1)
      const T draw = T(1) + psi;
      const T d = draw < floor_d ? floor_d : draw;
      if (MODE == kPushReal && alive && draw < floor_d) ++nclamp;
      const T id = T(1) / d;
      const T gam = (T(1) + ux * ux + uy * uy + d * d) * T(0.5) * id;
      T f[5];
      f[0] = -ux * id * inv_hx;
      f[1] = -uy * id * inv_hy;
      if constexpr (MODE == kPushTrial) {   // the Bx/By kick is added below
        f[2] = gam * id * e1 + bz * uy * id;
        f[3] = gam * id * e2 - bz * ux * id;
      } else {
        f[2] = gam * id * e1 + by + bz * uy * id;
        f[3] = gam * id * e2 - bx - bz * ux * id;
      }
      f[4] = (ux * e1 + uy * e2) * id - ez;
      T y[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) y[c] = in.pk[c] - dz * (b0 * f[c]);
      if constexpr (MODE == kPushTrial) {
        const T cx = y[2], cy = y[3];
        const T kick = dz * b0;
        y[2] = cx - kick * by;
        y[3] = cy + kick * bx;
        if (a.rec) {   // what the later iterations of this slice start from
          const bool in_box = inside(ci0, fx0 + y[0], nx) && inside(cj0, fy0 + y[1], ny);
          const T dn = T(1) + y[4];
          const T idn = T(1) / (dn < floor_d ? floor_d : dn);
          T* r = a.rec;
          store_at(r, p, y[0]);
          store_at(r + np, p, y[1]);
          store_at(r + 2 * np, p, cx);
          store_at(r + 3 * np, p, cy);
          store_at(r + 4 * np, p, alive && in_box ? -w * idn : T(0));
          if constexpr (TAPE) store_at(r + 5 * np, p, y[4]);
        }
      }
      if (!alive) continue;
      if (!inside(ci0, fx0 + y[0], nx) || !inside(cj0, fy0 + y[1], ny)) {
        ++nabs;
        if (MODE == kPushReal) store_at(a.p.w, p, T(0));
        continue;
      }
      xi = y[0];
      eta = y[1];
      ux = y[2];
      uy = y[3];
      psi = y[4];
      if constexpr (MODE == kPushReal) {
        store_at(a.p.xi_x, p, xi);
        store_at(a.p.xi_y, p, eta);
        store_at(a.p.ux, p, ux);
        store_at(a.p.uy, p, uy);
        store_at(a.p.psi, p, psi);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          store_at(a.p.hist + ((a.k & 3) * 5 + c) * np, p, f[c]);
          store_at(a.p.pab + c * np, p, ab5_history(y[c], f[c], in.h[0][c], in.h[1][c], in.h[2][c], dz));
        }
      }
    } else if (!alive) {
      continue;
    }

    // deposit at the (new) position: rho - Jz = q w exactly, J = q w u / D
    const T draw = T(1) + psi;
    const bool clamped = draw < floor_d;
    const T d = clamped ? floor_d : draw;
    const T id = T(1) / d;
    const T omd = clamped ? T(1) - d : -psi;     // 1 - D
    double v[4];
    if (MODE == kPushTrial) {
      v[0] = static_cast<double>(-w * ux * id);
      v[1] = static_cast<double>(-w * uy * id);
    } else {
      const T u2 = ux * ux + uy * uy;
      const T uz = (u2 + omd * (T(1) + d)) * T(0.5) * id;
      v[0] = static_cast<double>(-w);
      v[1] = static_cast<double>(-w * ux * id);
      v[2] = static_cast<double>(-w * uy * id);
      v[3] = static_cast<double>(-w * uz * id);
    }
    deposit_particle<T, O, nch>(a.dep, tile, ts, ox, oy, nx, ny, tiled, owner, ci0, cj0, fx0, fy0,
                                xi, eta, v, nglob);
  }

  if (tiled) {
    __syncthreads();
    if (owner)
      flush_tile_owned<nch>(a.dep.ch, a.dep.sh, tile, ts, ox, oy, nx, ny);
    else
      flush_tile<nch>(a.dep.ch, tile, ts, ox, oy, nx, ny);
  }
  // counters (none of them is kept for a trial push)
  if constexpr (trial) return;
  const unsigned long long tc = block_sum(nclamp, red);
  const unsigned long long ta = block_sum(nabs, red);
  const unsigned long long tg = block_sum(nglob, red);
  if (threadIdx.x == 0) {
    if (tc) atomicAdd(&ctr->n_clamped, tc);
    if (MODE == kPushReal && ta) atomicAdd(&ctr->n_absorbed, ta);
    if (!trial && tg) atomicAdd(&ctr->n_dep_global, tg);
  }
}

// Sources of the explicit Bx/By solver for the particles of lattice tile
// (tbx, tby) at their slice-k state, in the final psi, Ez, Bz of slice k
// (shape order O >= 1).  Along the pusher's orbits (dx_p/dzeta = -u/D)
//   d_zeta J_perp = sum q w [ S d(u/D)/dzeta - (u/D) (grad_p S . u/D) ],
// whose B_perp part is -chi By (x) and +chi Bx (y) with chi = sum w S / D;
// the rest (DJx, DJy) and chi are deposited into dep.ch[0..2] = chi, DJx,
// DJy (FP64).  du/dzeta without B_perp: a_x = gamma/D (Ex-By) + Bz u_y/D,
// a_y = gamma/D (Ey+Bx) - Bz u_x/D; dPsi/dzeta = u.(E-vxB)_perp/D - Ez, and
// a floored D does not change.
template <typename T, int O>
__device__ __forceinline__ void explicit_tile(const Geom& g, const Lattice& L,
                                              const PushArgs<T>& a, int tbx, int tby,
                                              double* tile) {
  constexpr int nch = 3;
  const TileShape ts = tile_shape(L, a.tile_rows, a.tile_halo);
  const int ntile = ts.nw * ts.nh;
  const bool tiled = a.tiled != 0;
  const int I0 = tbx * ts.tx, J0 = tby * ts.ty;
  const int ox = (I0 >> ts.lpx) - ts.halo, oy = (J0 >> ts.lpy) - ts.halo;
  const int nx = g.nx, ny = g.ny;
  const double ihx = 1.0 / a.hx, ihy = 1.0 / a.hy;
  const T floor_d = static_cast<T>(a.psi_floor);
  // the first loads are in flight while the histogram is cleared
  ParticleLoad<T, kDepositOnly> in;
  in.load(L, a, ts, I0, J0, static_cast<int>(threadIdx.x));
  if (tiled) {
    __syncthreads();
    for (int e = threadIdx.x; e < nch * ntile; e += kBlock) tile[e] = 0.0;
    __syncthreads();
  }

  for (int e = threadIdx.x; e < ts.tx * ts.ty; e += kBlock) {
    if (e >= kBlock) in.load(L, a, ts, I0, J0, e);
    const int I = I0 + (e & (ts.tx - 1)), J = J0 + (e >> ts.ltx);
    const T w = in.w;
    T xi = in.y[0], eta = in.y[1];
    const T ux = in.y[2], uy = in.y[3], psi = in.y[4];
    pin(xi);
    pin(eta);
    const int ci0 = I >> ts.lpx, cj0 = J >> ts.lpy;
    const T fx0 = (T(2 * (I & (L.ppc_x - 1)) + 1)) / T(2 * L.ppc_x);
    const T fy0 = (T(2 * (J & (L.ppc_y - 1)) + 1)) / T(2 * L.ppc_y);
    int bi, bj;
    const T dx = shape::locate<O>(ci0, fx0 + xi, nx, bi);
    const T dy = shape::locate<O>(cj0, fy0 + eta, ny, bj);
    T e1, e2, ez, bz;
    if constexpr (O == 1) {
      Cic<T> cic;
      cic.at(bi, bj, dx, dy, nx, ny);
      auto n1 = cic.load(a.f.exmby), n2 = cic.load(a.f.eypbx), n3 = cic.load(a.f.ez), n4 = cic.load(a.f.bz);
      __builtin_amdgcn_sched_barrier(0);
      n1.pin();
      n2.pin();
      n3.pin();
      n4.pin();
      e1 = cic.sum(n1);
      e2 = cic.sum(n2);
      ez = cic.sum(n3);
      bz = cic.sum(n4);
    } else {
      T wx[O + 1], wy[O + 1];
      int ix[O + 1], iy[O + 1];
      bool okx[O + 1], oky[O + 1];
      shape::weights<O>(dx, wx);
      shape::weights<O>(dy, wy);
      shape::axis_nodes<O>(bi, nx, ix, okx);
      shape::axis_nodes<O>(bj, ny, iy, oky);
#pragma unroll
      for (int q = 0; q <= O; ++q) {
        wx[q] = okx[q] ? wx[q] : T(0);
        wy[q] = oky[q] ? wy[q] : T(0);
      }
      e1 = shape::interp<O>(a.f.exmby, ix, iy, wx, wy, nx);
      e2 = shape::interp<O>(a.f.eypbx, ix, iy, wx, wy, nx);
      ez = shape::interp<O>(a.f.ez, ix, iy, wx, wy, nx);
      bz = shape::interp<O>(a.f.bz, ix, iy, wx, wy, nx);
    }
    if (w == T(0)) continue;
    const T draw = T(1) + psi;
    const bool clamped = draw < floor_d;
    const T d = clamped ? floor_d : draw;
    const T id = T(1) / d;
    const T gam = (T(1) + ux * ux + uy * uy + d * d) * T(0.5) * id;
    const T ax = gam * id * e1 + bz * uy * id;
    const T ay = gam * id * e2 - bz * ux * id;
    const T apsi = clamped ? T(0) : (ux * e1 + uy * e2) * id - ez;
    const T qn = -w;
    const double cx = static_cast<double>(qn * (ax * id - ux * apsi * id * id));
    const double cy = static_cast<double>(qn * (ay * id - uy * apsi * id * id));
    const double vx = static_cast<double>(ux * id), vy = static_cast<double>(uy * id);
    const double qd = static_cast<double>(qn);
    const double chi_p = static_cast<double>(w * id);
    double sx[O + 1], sy[O + 1], gx[O + 1], gy[O + 1];
    shape::weights<O>(static_cast<double>(dx), sx);
    shape::weights<O>(static_cast<double>(dy), sy);
    shape::weight_slopes<O>(static_cast<double>(dx), gx);
    shape::weight_slopes<O>(static_cast<double>(dy), gy);
    const int li = bi - ox, lj = bj - oy;
    const bool in_tile = tiled && li >= 0 && li + O < ts.nw && lj >= 0 && lj + O < ts.nh;
#pragma unroll
    for (int qb = 0; qb <= O; ++qb) {
      const int gj = bj + qb;
#pragma unroll
      for (int qa = 0; qa <= O; ++qa) {
        const int gi = bi + qa;
        const double sw = sx[qa] * sy[qb];
        const double vg = vx * (gx[qa] * sy[qb] * ihx) + vy * (sx[qa] * gy[qb] * ihy);
        const double v0 = chi_p * sw;
        // (u/D) dS/dzeta with dS/dzeta = -(grad_p S . u/D) = -vg
        const double v1 = cx * sw - qd * vx * vg;
        const double v2 = cy * sw - qd * vy * vg;
        if (in_tile) {
          double* t = tile + (lj + qb) * ts.nw + (li + qa);
          lds_add(t, v0);
          lds_add(t + ntile, v1);
          lds_add(t + 2 * ntile, v2);
        } else if (gi >= 1 && gi < nx && gj >= 1 && gj < ny) {
          const size_t o = static_cast<size_t>(gj) * nx + gi;
          global_add(a.dep.ch[0] + o, v0);
          global_add(a.dep.ch[1] + o, v1);
          global_add(a.dep.ch[2] + o, v2);
        }
      }
    }
  }

  if (tiled) {
    __syncthreads();
    flush_tile<nch>(a.dep.ch, tile, ts, ox, oy, nx, ny);
  }
}

}  // namespace push_detail
}  // namespace qsp
