// Batched 2D Dirichlet Poisson / Helmholtz solves with type-I sine transforms
// (fast Poisson solver of HiPACE++, arXiv:2109.10277 Sec. III.B), written for
// gfx950: every 1D transform runs inside LDS.
//
// Three passes per solve:
//   P1 (row pass)     source assembly (FP64 deposits -> T) fused with the
//                      forward DST along x, one workgroup per block of rows;
//   P2 (column pass)   forward DST along y, division by the eigenvalues of
//                      (lap_h - shift), inverse DST along y (plus an optional
//                      -d_y of the result), one workgroup per column strip;
//   P3 (row pass)     inverse DST along x with a fused epilogue (plain store,
//                      -d_x for Ex-By, or the predictor-corrector update with
//                      its FP64 residual reduction).
//
// Transform used (per row x_0..x_{n-1}, x_0 = x_n = 0):
//   S_p = sum_j x_j sin(pi j p / n); inverse x = (2/n) S(S(x)), the 2D factor
//   4/(nx ny) folded into the eigenvalue division of P2.  Three cores, chosen
//   by the row length (sym_core, wave_core in common.hpp): a matrix product
//   for 16 to 64 points (FP32: 128), complex FFTs of the odd extension for the others.
#pragma once

#include <stdexcept>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "partials.hpp"

namespace qsp {
namespace dst_detail {

template <typename T>
__device__ inline Cplx<T> cmul(Cplx<T> a, Cplx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

// Orders the LDS accesses of one wavefront: they execute in order, so an
// exchange inside a wave only needs the compiler kept from reordering them.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keeps a loaded value in its register from here on: without it the compiler
// moves a load whose value only feeds a select into a branch beside the
// select, and so turns a batch of loads into one memory round trip each
// (source assembly of a 1024^2 corrector pass, FP32: 31.2k of the kernel's
// 41k cycles in three dependent round trips per element).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

template <typename T>
__device__ inline Cplx<T> cadd(Cplx<T> a, Cplx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__device__ inline Cplx<T> csub(Cplx<T> a, Cplx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T>
__device__ inline Cplx<T> cmul_mi(Cplx<T> a) { return {a.im, -a.re}; }   // -i a

// in-place DFT of length 4 (forward)
template <typename T>
__device__ __forceinline__ void dft4(Cplx<T>& y0, Cplx<T>& y1, Cplx<T>& y2, Cplx<T>& y3) {
  const Cplx<T> c0 = cadd(y0, y2), c1 = csub(y0, y2), c2 = cadd(y1, y3);
  const Cplx<T> c3 = cmul_mi(csub(y1, y3));
  y0 = cadd(c0, c2);
  y2 = csub(c0, c2);
  y1 = cadd(c1, c3);
  y3 = csub(c1, c3);
}

// in-place DFT of length 8 (forward), natural order in and out
template <typename T>
__device__ __forceinline__ void dft8(Cplx<T>* v) {
  const T h = T(0.70710678118654752440);
  Cplx<T> a[4], b[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    a[m] = cadd(v[m], v[m + 4]);
    b[m] = csub(v[m], v[m + 4]);
  }
  // b_m *= e^{-2 pi i m / 8}
  b[1] = {h * (b[1].re + b[1].im), h * (b[1].im - b[1].re)};
  b[2] = cmul_mi(b[2]);
  b[3] = {h * (b[3].im - b[3].re), -h * (b[3].re + b[3].im)};
  dft4(a[0], a[1], a[2], a[3]);
  dft4(b[0], b[1], b[2], b[3]);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[2 * r] = a[r];
    v[2 * r + 1] = b[r];
  }
}

// ---------------------------------------------------------------------------
// FP32 core for n = 256 and 512, without a recurrence (a half-length FFT with
// a prefix sum for the odd outputs loses ~1e-4 of Ey+Bx at 512^2-1024^2 through
// the centred differences taken of the solved fields).  The two
// rows a, b of a pair are extended oddly to length N = 2n (z_j = a_j + i b_j,
// z_{2n-j} = -z_j, z_0 = z_n = 0) and transformed by one complex FFT of
// length N: with X = DFT_N(z), S^a_p = -Im X_p / 2 and S^b_p = Re X_p / 2.
// Every output carries plain FFT round-off.
//
// One wave per pair, N = 64 P (P = 8, 16 points per lane), as a 4-step
// FFT with the index j = l + 64 m (lane l, register m) and k = k1 + P k2:
//   A   each lane: DFT_P over m in registers, times W_N^{l k1};
//   B1  DFT_64 over l split as 8 x 8 (l = la + 8 lb, k2 = c1 + 8 c2):
//       DFT_8 over lb, times W_64^{la c1};
//   B2  DFT_8 over la.
// Two transposes through the pair's LDS region (rows of 72 complex per k1:
// the transposes and the strided DFT_8 reads touch every bank once per two
// rows), no workgroup barrier.
// ---------------------------------------------------------------------------
constexpr int kCorePitch = 72;   // complex entries per k1 row of the transposes

// Row layout in LDS around the two FFT cores (gfx950 serves LDS as 32 banks
// of 4 bytes, half a wave of 4-byte or a quarter of 8-byte accesses at a
// time): 4 padding words after every 32.  Row b of a pair lies at an offset
// = 4 (mod 32) words (8 from 1024 points up), pairs 8 (mod 32) apart with the
// wave core, 16 with the symmetric core.  Then the cores' last-stage writes
// (k = k1 + 16 c1 or kb + P c1 + const over the lanes) land on distinct banks,
// and so do the column pass's strip accesses; runs of 32 consecutive words
// (row passes, the first stage) stay contiguous.
template <typename T>
struct CoreLay {
  static constexpr int S = sizeof(T) == 4 ? 5 : 4;   // log2 of the run
  static constexpr int Q = sizeof(T) == 4 ? 4 : 2;   // padding after it
  __host__ __device__ static constexpr int ridx(int i) { return i + Q * (i >> S); }
  __host__ __device__ static constexpr int rlen(int n) {
    return ((ridx(n) + 31) & ~31) + (n >= 1024 ? 8 : 4);
  }
  __host__ __device__ static constexpr int rpos(int n, int pitch, int r, int i) {
    return (r >> 1) * pitch + (r & 1) * rlen(n) + ridx(i);
  }
};

// W_32^k = e^{-2 pi i k / 32} for k >= 0 (from cos(2 pi k / 32), k = 0..8;
// W_32^{k+16} = -W_32^k).  Called with compile-time k only.
template <typename T>
__device__ __forceinline__ Cplx<T> w32(int k) {
  constexpr double c32[9] = {1.0,
                             0.98078528040323044913,
                             0.92387953251128675613,
                             0.83146961230254523708,
                             0.70710678118654752440,
                             0.55557023301960222474,
                             0.38268343236508977173,
                             0.19509032201612826785,
                             0.0};
  const double sg = (k & 16) ? -1.0 : 1.0;
  k &= 15;
  const double c = k <= 8 ? c32[k] : -c32[16 - k];
  const double s = k <= 8 ? c32[8 - k] : c32[k - 8];
  return {static_cast<T>(sg * c), static_cast<T>(-sg * s)};
}

// In-register forward DFT of length P = R1 * 8 (R1 = 1, 2), in place with
// j = j0 + 8 j1 and k = k0 + R1 k1: DFT_R1 over j1, twiddles W_P^{j0 k0},
// DFT_8 over j0.  X_k ends at position dft_pos<P>(k) = 8 k0 + k1.
template <int P>
__host__ __device__ constexpr int dft_pos(int k) {
  return 8 * (k % (P / 8)) + k / (P / 8);
}

template <int P, typename T>
__device__ __forceinline__ void dft_reg(Cplx<T>* v) {
  constexpr int R1 = P / 8;
  static_assert(R1 == 1 || R1 == 2, "8 or 16 points");
  if constexpr (R1 == 2) {
#pragma unroll
    for (int j0 = 0; j0 < 8; ++j0) {
      const Cplx<T> a = v[j0], b = v[j0 + 8];
      v[j0] = cadd(a, b);
      v[j0 + 8] = csub(a, b);
    }
  }
  if constexpr (R1 > 1) {
#pragma unroll
    for (int k0 = 1; k0 < R1; ++k0)
#pragma unroll
      for (int j0 = 1; j0 < 8; ++j0) v[8 * k0 + j0] = cmul(v[8 * k0 + j0], w32<T>(j0 * k0 * (32 / P)));
  }
#pragma unroll
  for (int k0 = 0; k0 < R1; ++k0) dft8(v + 8 * k0);
}

// DST-I of one pair (rows a at g, b at g + rlen(n), entry 0 = 0) by one
// wave, in place; twa[k1 - 1] = W_N^{l k1} (the lane's registers), w64[la * 9
// + c1] = W_64^{la c1} (LDS).  The pair's region holds P rows of kCorePitch
// complex.
// Output scaling of the core: none (plain transform).  The cores call
// epi(q, oa, ob) for their q-th output slot of the lane.
struct NoScale {
  template <typename T>
  __device__ void operator()(int, T&, T&) const {}
};

// 1 / d: the hardware estimate in FP32 (1 ulp), refined by two Newton steps
// in FP64, which need a finite d
__device__ __forceinline__ float recip(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double recip(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(fma(-d, y, 1.0), y, y);
  return fma(fma(-d, y, 1.0), y, y);
}

// Output scaling of the core in the column pass: S_k of the pair's columns
// p_a, p_b divided by (lambda_x(p) + lambda_y(k) - shift) nx ny / 4, the
// eigenvalue of the shifted Laplacian times the two transforms'
// normalisation; column p = 0 (a boundary node line) is zero.  ry holds
// (lambda_y(k) - shift) nx ny / 4 for the lane's NK output slots k (see
// core_out_k, sym_out_k), xa / xb lambda_x(p) nx ny / 4, in FP64 held to a
// quarter of the range where their sum might not be finite (eigen_range).
// Shorter FP32 columns add FP32 terms, and FP64 columns multiply by the
// reciprocal: with a division solves of 1024 x 512 points err no less (4.6e-16
// against 4.5e-16) and take 41.1 us instead of 40.1, the 512^2 FP64 box 30.4 ms
// instead of 29.8.
// Whether the terms may reach 2^1022 (spacings or a shift at the end of the
// range); tested once, under the strip load: holding the terms always took the
// 512^2 FP64 column pass from 12.55 to 12.65 us.
__device__ __forceinline__ bool eigen_range(const Geom& g, double shift, double inorm) {
  const double hx2 = g.hx * g.hx, hy2 = g.hy * g.hy;
  return !(4.0 * inorm < 0x1p1000 * hx2 && 4.0 * inorm < 0x1p1000 * hy2 && shift * inorm < 0x1p1000);
}
template <typename T, int NK>
struct EigenScale {
  T ry[NK];
  T xa, xb;
  bool za;
  __device__ void operator()(int q, T& oa, T& ob) const {
    const T ra = recip(xa + ry[q]);
    const T rb = recip(xb + ry[q]);
    oa = za ? T(0) : oa * ra;
    ob *= rb;
  }
};

// The same for FP32 columns of 2048 points, the sum formed in FP64, rounded
// once and divided by: terms rounded before the sum and the reciprocal err up
// to 6 units of 2^-24 there instead of 3.  The outputs of a lane are k0 + 256 q
// (or 4096 less that), so lambda_y = -2 / h^2 + c cos(pi q / 8) + s sin(pi q / 8)
// with c = lambda_y(k0) + 2 / h^2 and s = lambda_y(k0 + 1024) + 2 / h^2: four
// doubles instead of sixteen, exact to 1e-10 of the smallest eigenvalue.  2048^2
// nodes, three fields: 126 us; 153 with sixteen doubles a lane (191 registers
// against 165, two waves a SIMD instead of three), 130 with rounded terms.
template <typename T, int N>
constexpr bool eigen_once = sizeof(T) == 4 && N > 1024;
struct EigenOnce {
  double c, s;     // times nx ny / 4
  double xa, xb;   // (lambda_x(p) - shift - 2 / h^2) nx ny / 4
  bool za;
  __device__ void operator()(int q, float& oa, float& ob) const {
    const Cplx<double> w = w32<double>(2 * q);   // cos, -sin (pi q / 8)
    const double y = c * w.re - s * w.im;
    oa = za ? 0.f : oa / static_cast<float>(xa + y);
    ob /= static_cast<float>(xb + y);
  }
};

// Output slots of a lane of the wave core (P points per lane, lane l):
// k = (l >> 3) + 8 t + P (l & 7) + 8 P c2 in slot q = 4 t + c2.
template <int P>
__device__ __forceinline__ int core_out_k(int l, int q) {
  return (l >> 3) + 8 * (q >> 2) + P * (l & 7) + 8 * P * (q & 3);
}

template <int P, typename Epi = NoScale>
__device__ __forceinline__ void wave_dst_core(float* g, const Cplx<float> (&twa)[P - 1],
                                              const Cplx<float>* w64,
                                              const Epi& epi = Epi{}) {
  using Pd = CoreLay<float>;
  constexpr int n = 32 * P;
  constexpr int NB = P / 8;
  const int l = threadIdx.x & 63;
  float* ra = g;
  float* rb = g + Pd::rlen(n);
  Cplx<float>* s = reinterpret_cast<Cplx<float>*>(g);
  // A: z_{l + 64 m}; m >= P/2 from the mirror 2n - j = 64 (P - m) - l
  Cplx<float> v[P];
#pragma unroll
  for (int m = 0; m < P / 2; ++m) {
    const int j = Pd::ridx(l + 64 * m);
    v[m] = {ra[j], rb[j]};
  }
#pragma unroll
  for (int m = P / 2; m < P; ++m) {
    const int jm = 64 * (P - m) - l;          // in [1, n], n only for l = 0, m = P/2
    const int j = Pd::ridx(jm < n ? jm : 0);
    const float fa = ra[j], fb = rb[j];
    v[m] = {jm < n ? -fa : 0.f, jm < n ? -fb : 0.f};
  }
  wave_sync();
  dft_reg<P>(v);
#pragma unroll
  for (int k1 = 0; k1 < P; ++k1) {
    const Cplx<float> y = v[dft_pos<P>(k1)];
    s[k1 * kCorePitch + l] = k1 ? cmul(y, twa[k1 > 0 ? k1 - 1 : 0]) : y;
  }
  wave_sync();
  // B1: combos (k1, la) = (l >> 3 + 8 t, l & 7)
  const int la = l & 7, kb = l >> 3;
  Cplx<float> u[NB][8];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const Cplx<float>* r = s + (kb + 8 * t) * kCorePitch + la;
#pragma unroll
    for (int lb = 0; lb < 8; ++lb) u[t][lb] = r[8 * lb];
  }
  Cplx<float> wl[8];
  wl[0] = {1.f, 0.f};
#pragma unroll
  for (int c1 = 1; c1 < 8; ++c1) wl[c1] = w64[la * 9 + c1];
  wave_sync();
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    dft8(u[t]);
    Cplx<float>* r = s + (kb + 8 * t) * kCorePitch + la * 9;
    r[0] = u[t][0];
#pragma unroll
    for (int c1 = 1; c1 < 8; ++c1) r[c1] = cmul(u[t][c1], wl[c1]);
  }
  wave_sync();
  // B2: combos (k1, c1) = (l >> 3 + 8 t, l & 7); DFT_8 over la
  const int c1 = l & 7;
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const Cplx<float>* r = s + (kb + 8 * t) * kCorePitch + c1;
#pragma unroll
    for (int a = 0; a < 8; ++a) u[t][a] = r[a * 9];
  }
  wave_sync();
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    dft8(u[t]);
    const int k0 = kb + 8 * t + P * c1;       // k = k0 + 8 P c2, < n for c2 < 4
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {
      const int k = k0 + 8 * P * c2;
      const int j = Pd::ridx(k);
      float oa = -0.5f * u[t][c2].im, ob = 0.5f * u[t][c2].re;
      epi(4 * t + c2, oa, ob);
      ra[j] = k ? oa : 0.f;
      rb[j] = k ? ob : 0.f;
    }
  }
  wave_sync();
}

// ---------------------------------------------------------------------------
// Symmetric core (n = 128 .. 2048, FP32 and FP64): the FFT of the odd
// extension z (length N = 2n, rows a + i b) without its redundant half.  With
// H = n / 16, l = 0 .. 2H - 1, j = l + 2H m, k = k1 + 16 k2 the four-step FFT is
//   A_k1(l) = DFT_16 over m of z_{l + 2H m},  y_k1(l) = W_N^{l k1} A_k1(l),
//   X_{k1 + 16 k2} = DFT_2H over l of y_k1.
// z_{N-j} = -z_j gives y_k1(2H - l) = -conj(W_N^{l k1}) A_{16-k1}(l), so lanes
// l < H supply both ends of every row, and X_{N-k} = -X_k lets the rows
// k1 = 0 .. 8 give every output (k >= n as -X at N - k).  A wave of 64 lanes
// transforms a pair at n = 1024 where the full extension takes two, and the
// LDS exchanges, which bound the 1024^2 passes (13.6k of the 21.5k cycles of a
// column pass were LDS issue), move 9/16 of the data.
//   A    main lane l (H per pair): DFT_16, 9 rows x 2 ends;
//        l = H, its own mirror image: y_k1(H) = -2i sum_{m<8} z_{H + 2H m}
//        sin(pi (2m + 1) k1 / 16), by lanes of the next wave;
//   --   workgroup barrier;
//   B    row k1 by G = H / 8 lanes of 16 points (rows 0-7: the main lanes, row
//        8: the next wave): DFT_16 over l = g + G lb, W_2H^{g c1}, exchange
//        inside the row, DFT_G; k2 = c1 + 16 c2.  At n = 128 a lane holds a
//        whole row.
// The rows of the exchange region are RP = 16 (G + 1) + G complex apart and
// the exchange entries G + 1: every access pattern (consecutive l; g + G lb
// over rows; c1 (G + 1) + g) meets each bank once per service group.
// The twiddles of stage A stay in the lane's registers, those of stage B (16 G,
// rows of 17) in LDS, so a transform issues no global load.  (All of them and
// the column pass's eigenvalues by global loads of every lane moved 80 KB a
// workgroup through the vector cache, five times its strip.)
// ---------------------------------------------------------------------------
template <int LOGN, int NP = 1>
struct Sym {
  static constexpr int n = 1 << LOGN;
  static constexpr int H = n / 16, NL = 2 * H;
  static constexpr int G = sym_g(n);
  static constexpr int GP = G + 1;
  static constexpr int RP = G == 1 ? NL + 1 : 16 * GP + (G < 16 ? G : 0);
  static constexpr int pairs = NP;                         // per workgroup
  static constexpr int nmain = pairs * H;                  // main lanes
  static constexpr int xtra = (nmain + 63) / 64 * 64;      // first lane of the next wave
  static_assert(H >= 8 && xtra + 64 <= kBlock && 16 * pairs <= 64, "workgroup shape");
  // T units in front of the exchange region, and of a whole pair
  template <typename T>
  __host__ __device__ static constexpr int soff() {
    return (CoreLay<T>::rlen(n) + CoreLay<T>::ridx(n) + 31) & ~31;
  }
  template <typename T>
  __host__ __device__ static constexpr int pitch() {
    return ((soff<T>() + 2 * 9 * RP + 31) & ~31) + 16;
  }
};

// A lane's tasks: stage A of row l (main) or the l = H entry k1 (next wave),
// stage B of row k1 with position g in it.
template <int LOGN, int NP>
struct SymLane {
  using Y = Sym<LOGN, NP>;
  bool main, mid, row;   // has a main stage A, a middle entry, a row of stage B
  int pair_a, l;         // stage A (l = entry k1 for a middle lane)
  int pair_b, k1, g;     // stage B
  __device__ SymLane() {
    const int L = static_cast<int>(threadIdx.x), x = L - Y::xtra;
    main = L < Y::nmain;
    mid = x >= 0 && x < 16 * Y::pairs && (x & 15) < 9;
    row = main || (x >= 0 && x < Y::G * Y::pairs);
    pair_a = main ? L / Y::H : (mid ? x >> 4 : 0);
    l = main ? L % Y::H : (mid ? x & 15 : 0);
    pair_b = main ? L / Y::H : (row ? x / Y::G : 0);
    k1 = main ? (L % Y::H) / Y::G : 8;
    g = main ? L % Y::G : (row ? x % Y::G : 0);
  }
};

template <typename T, int LOGN>
struct SymTw {
  Cplx<T> a[8];        // W_N^{l k}, k = 1..8; middle lane: sines in re
  Cplx<T> b;           // the thread's entry of the stage-B table
};
template <typename T, int LOGN, int NP>
__device__ __forceinline__ SymTw<T, LOGN> sym_load(const Cplx<T>* __restrict__ tw) {
  using Y = Sym<LOGN, NP>;
  const SymLane<LOGN, NP> q;
  SymTw<T, LOGN> w;
  // table entries of the lane: row strides H (main) or 1 (a middle entry's sines)
  const Cplx<T>* pa = q.main ? tw + Y::H + q.l : tw + sym_table_s(Y::n) + 8 * q.l;
  const int st = q.main ? Y::H : 1;
#pragma unroll
  for (int k = 0; k < 8; ++k) w.a[k] = pa[k * st];
  const int tid = static_cast<int>(threadIdx.x);
  w.b = tw[sym_table_w(Y::n) + (tid < 16 * Y::G ? tid : 0)];
  return w;
}

// Output k of slot q of a lane's row, and whether the slot's value is stored
// (rows 0 and 8 hold every value twice).
template <int LOGN, int NP>
__device__ __forceinline__ int sym_out_k(const SymLane<LOGN, NP>& t, int q, bool& stored) {
  using Y = Sym<LOGN, NP>;
  const int c1 = Y::G > 1 ? t.g + Y::G * (q / Y::G) : q;
  const int k2 = Y::G > 1 ? c1 + 16 * (q % Y::G) : q;
  const bool direct = k2 < Y::H;
  stored = direct || (t.k1 & 7) != 0;
  return direct ? t.k1 + 16 * k2 : 16 * (Y::NL - k2) - t.k1;
}

template <typename B, typename T>
__device__ __forceinline__ Cplx<B> widen(const Cplx<T>& a) {
  return {static_cast<B>(a.re), static_cast<B>(a.im)};
}
template <typename T, typename B>
__device__ __forceinline__ Cplx<T> narrow(const Cplx<B>& a) {
  return {static_cast<T>(a.re), static_cast<T>(a.im)};
}

// Transform of the workgroup's pairs in place (entry 0 of every row = 0 on
// entry; S_k on exit, entry 0 = 0).  Every thread of the workgroup calls it;
// the caller synchronises before the rows are read again.  epi(q, oa, ob)
// sees the values of slot q.  A and B are the types the two stages sum in.
// The forward transforms sum FP32 rows in FP64 registers (the exchange stays
// in T): a mirrored value carries the round-off of the value it copies, so the
// low modes' errors add up where independently formed halves partly cancel,
// and psi of a 1024^2 box with random beams erred 8.6e-7 against 5.9e-7 with
// the whole 2n-point FFT.  With FP64 sums 5.96e-7, every other field below
// what it was; the box takes 100.3 ms against 97.6 with FP32 sums and 107.2
// with the whole FFT.  FP64 in stage A alone: 6.06e-7, 98.1 ms; in stage B
// alone 8.5e-7; in the inverse transforms too 5.9e-7, 106.5 ms.
template <typename T, typename A, typename B, int LOGN, int NP, typename Epi = NoScale>
__device__ __forceinline__ void sym_dst(T* buf, const SymTw<T, LOGN>& w, const Cplx<T>* tb,
                                        const Epi& epi = Epi{}) {
  using Y = Sym<LOGN, NP>;
  using Pd = CoreLay<T>;
  constexpr int n = Y::n, H = Y::H, NL = Y::NL, G = Y::G, RP = Y::RP;
  const SymLane<LOGN, NP> t;
  {
    const T* ra = buf + t.pair_a * Y::template pitch<T>();
    const T* rb = ra + Pd::rlen(n);
    Cplx<T>* s = reinterpret_cast<Cplx<T>*>(buf + t.pair_a * Y::template pitch<T>() +
                                            Y::template soff<T>());
    if (t.main) {
      const int l = t.l;
      Cplx<A> v[16];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int j = Pd::ridx(l + NL * m);
        v[m] = {static_cast<A>(ra[j]), static_cast<A>(rb[j])};
      }
#pragma unroll
      for (int m = 8; m < 16; ++m) {
        const int jm = NL * (16 - m) - l;       // in [1, n], n only for l = 0, m = 8
        const int j = Pd::ridx(jm < n ? jm : 0);
        const T fa = ra[j], fb = rb[j];
        v[m] = {static_cast<A>(jm < n ? -fa : T(0)), static_cast<A>(jm < n ? -fb : T(0))};
      }
      dft_reg<16>(v);
      // both ends of every row (the mirror end of l = 0 falls on the unused
      // entry NL of the row)
      s[l] = narrow<T>(v[dft_pos<16>(0)]);
      s[NL - l] = narrow<T>(Cplx<A>{-v[dft_pos<16>(0)].re, -v[dft_pos<16>(0)].im});
#pragma unroll
      for (int k = 1; k <= 8; ++k) {
        const Cplx<A> c = {static_cast<A>(w.a[k - 1].re), static_cast<A>(w.a[k - 1].im)};
        s[k * RP + l] = narrow<T>(cmul(v[dft_pos<16>(k)], c));
        const Cplx<A> m = cmul(v[dft_pos<16>(16 - k)], Cplx<A>{c.re, -c.im});
        s[k * RP + NL - l] = narrow<T>(Cplx<A>{-m.re, -m.im});
      }
    } else if (t.mid) {
      A sa = A(0), sb = A(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int j = Pd::ridx(H + NL * m);
        sa += static_cast<A>(ra[j]) * w.a[m].re;
        sb += static_cast<A>(rb[j]) * w.a[m].re;
      }
      s[t.l * RP + H] = narrow<T>(Cplx<A>{A(2) * sb, A(-2) * sa});
    }
  }
  __syncthreads();
  if (!t.row) return;
  T* ra = buf + t.pair_b * Y::template pitch<T>();
  T* rb = ra + Pd::rlen(n);
  Cplx<T>* s = reinterpret_cast<Cplx<T>*>(ra + Y::template soff<T>()) + t.k1 * RP;
  auto put = [&](int q, const Cplx<B>& value) {
    const Cplx<T> X = narrow<T>(value);
    bool stored;
    const int k = sym_out_k(t, q, stored);
    const int c1 = G > 1 ? t.g + G * (q / G) : q;
    const int k2 = G > 1 ? c1 + 16 * (q % G) : q;
    T oa = k2 < H ? T(-0.5) * X.im : T(0.5) * X.im;
    T ob = k2 < H ? T(0.5) * X.re : T(-0.5) * X.re;
    epi(q, oa, ob);
    if (stored) {
      const int j = Pd::ridx(k);
      ra[j] = k ? oa : T(0);
      rb[j] = k ? ob : T(0);
    }
  };
  Cplx<B> x[16];
#pragma unroll
  for (int lb = 0; lb < 16; ++lb) x[lb] = widen<B>(s[t.g + G * lb]);
  Cplx<T> wb[G > 1 ? 15 : 1];
  if constexpr (G > 1) {
#pragma unroll
    for (int c = 1; c < 16; ++c) wb[c - 1] = tb[17 * t.g + c];
  }
  dft_reg<16>(x);
  if constexpr (G == 1) {
#pragma unroll
    for (int q = 0; q < 16; ++q) put(q, x[dft_pos<16>(q)]);
  } else {
    wave_sync();
#pragma unroll
    for (int c = 0; c < 16; ++c)
      s[c * Y::GP + t.g] = narrow<T>(c ? cmul(x[dft_pos<16>(c)], widen<B>(wb[c > 0 ? c - 1 : 0])) : x[dft_pos<16>(0)]);
    wave_sync();
#pragma unroll
    for (int si = 0; si < 16 / G; ++si) {
      const Cplx<T>* r = s + (t.g + G * si) * Y::GP;
      Cplx<B> u[G];
#pragma unroll
      for (int a = 0; a < G; ++a) u[a] = widen<B>(r[a]);
      if constexpr (G == 2) {
        const Cplx<B> u0 = u[0];
        u[0] = cadd(u0, u[1]);
        u[1] = csub(u0, u[1]);
      } else if constexpr (G == 4) {
        dft4(u[0], u[1], u[2], u[3]);
      } else if constexpr (G == 8) {
        dft8(u);
      } else {
        dft_reg<16>(u);
      }
#pragma unroll
      for (int c2 = 0; c2 < G; ++c2) put(G * si + c2, u[G == 16 ? dft_pos<16>(c2) : c2]);
    }
  }
}

// ---------------------------------------------------------------------------
// Matrix core (n = 16 to 64, in FP32 128): the transform of 16 rows as a
// product with the sine matrix on the matrix cores (16x16x4).  The inverse
// transforms sum in FP64 in both precisions: independently rounded FP32 sums
// put white round-off on the solution, which the differences taken of it
// (Ex - By) amplify (1.5-2.5 times the error of a half-length FFT at 64^2 and
// 128^2); in front of the eigenvalue division, which damps it, FP32 sums do.
// Such rows are bound by the length of the chain, not by operations: one LDS
// read of the operand, at most 8 dependent matrix instructions (two chains of
// 16 at 128 points) and one LDS write take the place of a half-length FFT with
// its three exchanges and a prefix sum (64^2 in FP32: box 7.28 -> 4.42 ms, 4.54
// with all sums in FP64, 4.15 with none; errors at or below what they were,
// field by field).
// From 32 points up sin(pi (n - m) k / n) = -(-1)^k sin(pi m k / n) folds a row
// to f_m + f_{n-m} for the odd outputs and f_m - f_{n-m} for the even ones,
// m < n/2, with f_{n/2} in the place of the pair m = 0 (odd outputs only): each
// wave forms 16 outputs of one parity from n/2 products.
// A lane holds row l % 16 and the K/4 operands m = (K/4) (l / 16) + s, s < K/4,
// of step s, both of the rows and of the matrix, so it reads consecutive
// values of the rows (and gathers the matrix from a table of 2n sines, which
// the L1 holds): rows lie in LDS with f_m at m and f_{n-m} at n/2 + m (pos), 16 bytes
// of padding after each row, which puts a quarter wave's 16-byte reads on
// distinct banks.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mfma4(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kDenseRows = 16;   // rows (columns) per workgroup

template <typename T, int LOGN>
struct Dense {
  static constexpr int n = 1 << LOGN;
  static constexpr bool fold = dense_fold(n);
  static constexpr int KL = dense_lane(n);     // operands per lane
  static constexpr int NT = n / 16;            // tiles of 16 outputs
  static constexpr int TW = NT > 4 ? NT / 4 : 1;   // tiles per wave (both parities from two up)
  static constexpr int NW = NT / TW;           // busy waves
  static constexpr int pitch = n + 16 / static_cast<int>(sizeof(T));
  // sums of a transform: FP64, or with FWD (in front of the eigenvalue
  // division) the field's own precision
  template <bool FWD>
  using Sum = std::conditional_t<FWD, T, double>;
  template <bool FWD>
  using V4 = std::conditional_t<std::is_same_v<Sum<FWD>, float>, f32x4, f64x4>;
  __host__ __device__ static constexpr int ridx(int i) {
    return fold && i >= n / 2 ? n / 2 + ((n - i) & (n / 2 - 1)) : i;
  }
  __host__ __device__ static constexpr int rlen(int) { return pitch; }
  __host__ __device__ static constexpr int rpos(int, int, int r, int i) { return r * pitch + ridx(i); }
  // row of the 16x16 result that register r of a lane holds (column l % 16)
  template <bool FWD>
  __device__ static __forceinline__ int row_of(int lane, int r) {
    return std::is_same_v<Sum<FWD>, float> ? 4 * (lane >> 4) + r : (lane >> 4) + 4 * r;
  }
  // the lane's matrix operands: of one tile, of the wave's tiles
  static __device__ __forceinline__ void load_tile(const Cplx<T>* tw, int tile, double (&a)[KL]) {
    const int lane = static_cast<int>(threadIdx.x) & 63;
#pragma unroll
    for (int s = 0; s < KL; ++s)
      a[s] = load_at(reinterpret_cast<const double*>(tw), dense_angle(n, tile, lane, s));
  }
  struct Tab {
    double a[TW][KL];
  };
  static __device__ __forceinline__ Tab load(const Cplx<T>* tw) {
    Tab t;
    const int wave = static_cast<int>(threadIdx.x) >> 6;
#pragma unroll
    for (int q = 0; q < TW; ++q) load_tile(tw, wave < NW ? wave * TW + q : q, t.a[q]);
    return t;
  }
  // 16 outputs (of one parity with folded rows) of the 16 rows at f
  template <bool FWD>
  static __device__ __forceinline__ V4<FWD> product(const T* f, const double (&a)[KL], bool odd) {
    T v[KL], w[KL];
    fetch(f, v, w);
    return chain<FWD>(v, w, a, odd);
  }
  // the outputs of the wave's tiles of the rows at f
  template <bool FWD>
  static __device__ __forceinline__ void tiles_of(const T* f, const Tab& t, int wave, V4<FWD> (&acc)[TW]) {
    T v[KL], w[KL];
    fetch(f, v, w);
#pragma unroll
    for (int q = 0; q < TW; ++q) acc[q] = chain<FWD>(v, w, t.a[q], TW > 1 ? q & 1 : wave & 1);
  }
  static __device__ __forceinline__ void fetch(const T* f, T (&v)[KL], T (&w)[KL]) {
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const T* p = f + (lane & 15) * pitch + KL * (lane >> 4);
#pragma unroll
    for (int s = 0; s < KL; ++s) v[s] = p[s];
#pragma unroll
    for (int s = 0; s < KL; ++s) w[s] = fold ? p[n / 2 + s] : T(0);
  }
  template <bool FWD>
  static __device__ __forceinline__ V4<FWD> chain(const T (&v)[KL], const T (&w)[KL], const double (&a)[KL],
                                                  bool odd) {
    using S = Sum<FWD>;
    V4<FWD> acc = {S(0), S(0), S(0), S(0)};
#pragma unroll
    for (int s = 0; s < KL; ++s) {
      const S x = static_cast<S>(v[s]), y = static_cast<S>(w[s]);
      acc = mfma4(!fold ? x : odd ? x + y : x - y, static_cast<S>(a[s]), acc);
    }
    return acc;
  }
};

// One transform of the kDenseRows rows at buf; epi(slot, row, output, value)
// gives what is stored, slot = 0 .. 4 TW - 1 in order.  Output 0 is a product
// with zeros, which is not zero for an infinity or a NaN in the row, so the
// inverse transforms' epi stores its zero.  Ends without a barrier.
template <bool FWD, typename T, int LOGN, typename Epi>
__device__ __forceinline__ void dense_dst(T* buf, const typename Dense<T, LOGN>::Tab& t, Epi&& epi) {
  using D = Dense<T, LOGN>;
  const int wave = static_cast<int>(threadIdx.x) >> 6, lane = static_cast<int>(threadIdx.x) & 63;
  typename D::template V4<FWD> v[D::TW];
  if (wave < D::NW) D::template tiles_of<FWD>(buf, t, wave, v);
  __syncthreads();   // the rows are read
  if (wave < D::NW) {
#pragma unroll
    for (int q = 0; q < D::TW; ++q) {
      const int o = dense_out(D::n, wave * D::TW + q, lane & 15);
      T* out = buf + D::ridx(o);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = D::template row_of<FWD>(lane, r);
        out[row * D::pitch] = epi(4 * q + r, row, o, static_cast<T>(v[q][r]));
      }
    }
  }
}

// T units per row pair in LDS: the two padded rows with the matrix core, for
// the wave core the P rows of its transposes (laid over the rows), for the
// symmetric core the rows followed by its exchange region.
template <typename T>
__host__ __device__ constexpr int pair_pitch(int n) {
  if (sym_core(sizeof(T), n))
    return n == 128    ? Sym<7>::pitch<T>()
           : n == 256  ? Sym<8>::pitch<T>()
           : n == 512  ? Sym<9>::pitch<T>()
           : n == 1024 ? Sym<10>::pitch<T>()
                       : Sym<11>::pitch<T>();
  if (wave_core(sizeof(T), n)) return (n / 32) * kCorePitch * 2 + 8;   // = 8 (mod 32)
  return 2 * (n + 16 / static_cast<int>(sizeof(T)));
}

// Rows per workgroup of a row pass over rows of n values.  With the wave core
// two, one busy wave (more, smaller workgroups fill the chip).
template <typename T>
__host__ __device__ constexpr int pass_rows(int n) {
  return sym_core(sizeof(T), n) ? sym_rows(n) : (wave_core(sizeof(T), n) ? 2 : kDenseRows);
}

// The LDS row layout of a pass over rows of 2^LOGN values.
template <typename T, int LOGN>
using RowLay = std::conditional_t<sym_core(sizeof(T), 1 << LOGN) || wave_core(sizeof(T), 1 << LOGN),
                                  CoreLay<T>, Dense<T, LOGN>>;

// What a pass's transforms need besides the rows.  The tables' loads are
// issued when it is made (stage_tables), in front of the pass's own loads;
// commit() then writes to LDS what the transform reads there, after those
// loads, so that no wait for a table delays them.
//   symmetric core: the lane's stage-A twiddles in registers, stage B's in LDS
//   wave core:      the lane's W_N^{l k1} in registers, W_64 (72) in LDS
//   matrix core:    the lane's matrix operands in registers
template <int N>
struct WaveTw {
  Cplx<float> a[N / 32 - 1];   // k1 = 1 .. P - 1
  Cplx<float> w64;
};
template <typename T, int LOGN, int NP>   // NP: row pairs per workgroup (symmetric core)
struct Xform {
  static constexpr int n = 1 << LOGN;
  static constexpr bool sym = sym_core(sizeof(T), n), wav = wave_core(sizeof(T), n);
  unsigned char* lds;
  std::conditional_t<sym, SymTw<T, (LOGN >= 7 ? LOGN : 7)>,
                     std::conditional_t<wav, WaveTw<(wav ? n : 64)>,
                                        typename Dense<T, (LOGN <= 7 ? LOGN : 7)>::Tab>>
      w;
  // LDS places of the tables
  __device__ Cplx<T>* tw() const { return reinterpret_cast<Cplx<T>*>(lds); }
  __device__ __forceinline__ void commit() const {
    if constexpr (sym) {
      // the stage-B table, entry W_2H^{g c} at 17 g + c
      constexpr int NB = Sym<(sym ? LOGN : 7)>::G > 1 ? 16 * Sym<(sym ? LOGN : 7)>::G : 0;
      const int tid = static_cast<int>(threadIdx.x);
      if (tid < NB) tw()[17 * (tid >> 4) + (tid & 15)] = w.b;
    } else if constexpr (wav) {
      if (threadIdx.x < 72) tw()[threadIdx.x] = w.w64;
    }
  }
};

// Type-I sine transform of 2 NP rows of length n = 2^LOGN held in LDS; pair f
// = rows (2f, 2f+1) occupies buf[f*ppitch ..) (row 2f first, ppitch =
// pair_pitch(n)).  Entry 0 of every input row must be 0; on output entry p
// holds S_p (entry 0 = 0).  The wave core takes one pair per wave, the matrix
// core kDenseRows rows.  Ends with a workgroup barrier.
template <typename T, int LOGN, bool FWD, int NP>
__device__ __forceinline__ void block_dst(T* buf, int ppitch, const Xform<T, LOGN, NP>& x) {
  constexpr int n = 1 << LOGN;
  if constexpr (sym_core(sizeof(T), n)) {
    if constexpr (FWD)
      sym_dst<T, double, double, LOGN, NP>(buf, x.w, x.tw());
    else
      sym_dst<T, T, T, LOGN, NP>(buf, x.w, x.tw());
  } else if constexpr (wave_core(sizeof(T), n)) {
    const int wave = threadIdx.x >> 6;
    if (wave < NP) wave_dst_core<n / 32>(buf + static_cast<size_t>(wave) * ppitch, x.w.a, x.tw());
  } else {
    static_assert(2 * NP == kDenseRows, "rows of the matrix core");
    dense_dst<FWD, T, LOGN>(buf, x.w, [](int, int, int o, T v) { return FWD || o > 0 ? v : T(0); });
  }
  __syncthreads();
}

// Runs f(std::integral_constant<int, log2 n>) for the transform length n
// (a power of two in [16, 2048]); every kernel is instantiated per length.
template <typename F>
void with_logn(int n, F&& f) {
  switch (n) {
    case 16: f(std::integral_constant<int, 4>{}); break;
    case 32: f(std::integral_constant<int, 5>{}); break;
    case 64: f(std::integral_constant<int, 6>{}); break;
    case 128: f(std::integral_constant<int, 7>{}); break;
    case 256: f(std::integral_constant<int, 8>{}); break;
    case 512: f(std::integral_constant<int, 9>{}); break;
    case 1024: f(std::integral_constant<int, 10>{}); break;
    case 2048: f(std::integral_constant<int, 11>{}); break;
    default: throw std::invalid_argument("transform length must be a power of two in [16, 2048]");
  }
}

// Bytes of the per-axis tables a transform pass stages in LDS: the W_64 table
// (72 complex) of the wave core, the stage-B table of the symmetric core.
template <typename T>
__host__ __device__ constexpr size_t table_bytes(int n) {
  if (sym_core(sizeof(T), n))
    return static_cast<size_t>(sym_g(n) > 1 ? 17 * sym_g(n) : 0) * sizeof(Cplx<T>);
  return wave_core(sizeof(T), n) ? size_t(72) * sizeof(Cplx<T>) : 0;
}

// columns per column-pass workgroup: sym_cols with the symmetric core; four
// with the wave core, which makes the strip order of the intermediate planes
// possible (16-byte loads of whole strips; with two columns a lane's 8-byte
// segments took the pass 10.7 us at 512^2 in FP32, against 9.7, and twice the
// columns per workgroup 10.9); kDenseRows with the matrix core.
template <typename T>
__host__ __device__ constexpr int pass_cols(int ny) {
  return sym_core(sizeof(T), ny) ? sym_cols(ny) : (wave_core(sizeof(T), ny) ? 4 : kDenseRows);
}

// Issues the loads of an axis' transform tables for NP row pairs; the LDS part
// goes right after the workgroup's data region (Xform::commit).  Lanes without
// a part (and the wave and matrix cores' idle waves) load entry 0.
template <typename T, int LOGN, int NP>
__device__ __forceinline__ Xform<T, LOGN, NP> stage_tables(const AxisTables<T>& t, unsigned char* base) {
  constexpr int n = 1 << LOGN;
  Xform<T, LOGN, NP> x;
  x.lds = base;
  const int tid = static_cast<int>(threadIdx.x);
  if constexpr (sym_core(sizeof(T), n)) {
    x.w = sym_load<T, LOGN, NP>(t.tw);
  } else if constexpr (wave_core(sizeof(T), n)) {
#pragma unroll
    for (int k = 1; k < n / 32; ++k) x.w.a[k - 1] = t.tw[(tid >> 6) < NP ? k * 64 + (tid & 63) : 0];
    x.w.w64 = reinterpret_cast<const Cplx<T>*>(t.pre)[tid < 72 ? tid : 0];
  } else {
    x.w = Dense<T, LOGN>::load(t.tw);
  }
  return x;
}

// The tables of a row pass, placed after its rows.
template <typename T, int LOGN>
__device__ __forceinline__ auto stage_row_tables(const AxisTables<T>& t, unsigned char* smem_raw) {
  constexpr int n = 1 << LOGN, np = pass_rows<T>(n) / 2;
  return stage_tables<T, LOGN, np>(t, smem_raw + static_cast<size_t>(np) * pair_pitch<T>(n) * sizeof(T));
}
// LDS bytes of a pass over r rows (columns) of n values.
template <typename T>
constexpr size_t pass_lds(int r, int n) {
  return static_cast<size_t>(r / 2) * pair_pitch<T>(n) * sizeof(T) + table_bytes<T>(n);
}

// clears the planes of z, workgroup `bid` of `nblk` taking every nblk-th
// block of kBlock elements
__device__ __forceinline__ void zero_job(const ZeroJob& z, size_t bid, size_t nblk) {
  if (z.count == 0) return;
  const unsigned int n = static_cast<unsigned int>(z.n);
  const unsigned int stride = static_cast<unsigned int>(nblk) * kBlock;
  for (unsigned int i = static_cast<unsigned int>(bid) * kBlock + threadIdx.x; i < n; i += stride) {
#pragma unroll
    for (int c = 0; c < 8; ++c)   // plane pointers by constant index: kernel arguments
      if (c < z.count) store_at(z.p[c], i, 0.0);
  }
}

// The guess is loaded and stored in front of the pass's transform (up to kGuess
// elements a thread): behind it, its round trip came on top, and its stores
// now drain under the transform.
constexpr int kGuess = 6;
template <typename T>
struct GuessRegs {
  T x[kGuess], y[kGuess];
};

template <typename T>
__device__ __forceinline__ void guess_load(const GuessJob<T>& q, size_t n, size_t i0, size_t stride,
                                           GuessRegs<T>& g) {
  T x1[kGuess], x2[kGuess], y1[kGuess], y2[kGuess];
#pragma unroll
  for (int u = 0; u < kGuess; ++u) {
    const size_t i = i0 + u * stride;
    const size_t c = i < n ? i : 0;   // clamped: every load in bounds
    x1[u] = load_at(q.bx1, static_cast<unsigned int>(c));
    x2[u] = load_at(q.bx2, static_cast<unsigned int>(c));
    y1[u] = load_at(q.by1, static_cast<unsigned int>(c));
    y2[u] = load_at(q.by2, static_cast<unsigned int>(c));
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < kGuess; ++u) {
    g.x[u] = T(2) * x1[u] - x2[u];
    g.y[u] = T(2) * y1[u] - y2[u];
    pin(g.x[u]);
    pin(g.y[u]);
  }
}

template <typename T>
__device__ __forceinline__ void guess_store(const GuessJob<T>& q, size_t n, size_t i0, size_t stride,
                                            const GuessRegs<T>& g) {
#pragma unroll
  for (int u = 0; u < kGuess; ++u) {
    const size_t i = i0 + u * stride;
    if (i < n) {
      q.bx[i] = g.x[u];
      q.by[i] = g.y[u];
      if (q.tape_bx) {
        q.tape_bx[i] = g.x[u];
        q.tape_by[i] = g.y[u];
      }
    }
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Neighbouring column strips share cache lines, so strip s is given to
// the workgroup that lands on XCD (s / per) - keeping each XCD on one
// contiguous range of strips.
__device__ inline int xcd_strip(int b, int nstrip) {
  if (nstrip < 8 || (nstrip & 7)) return b;
  const int per = nstrip >> 3;
  return (b & 7) * per + (b >> 3);
}

// Workgroups per CU the transform kernels are compiled for: two (<= 256
// VGPRs) with the symmetric core, whose lanes keep 16 complex points and
// their twiddles, and FP32 rows of 128 points, whose lanes keep 32 matrix operands;
// four (<= 128 VGPRs) else, except the wave core's column pass, which keeps
// its eigenvalue divisors and a strip load in flight beside the core's
// registers.  The LDS of a CU (160 KiB) holds that many, but for FP64 rows of
// 1024 points (83,840 bytes a workgroup): one.
constexpr size_t kLdsPerCu = size_t(160) << 10;
constexpr int lds_blocks(int want, size_t lds) { return want * lds <= kLdsPerCu ? want : 1; }
constexpr size_t pass_lds_of(int logn, int tsize, bool rows) {
  const int n = 1 << logn;
  return tsize == 8 ? pass_lds<double>(rows ? pass_rows<double>(n) : pass_cols<double>(n), n)
                    : pass_lds<float>(rows ? pass_rows<float>(n) : pass_cols<float>(n), n);
}
constexpr int dst_blocks_per_cu(int logn, int tsize) {
  return lds_blocks(sym_core(tsize, 1 << logn) || logn == 7 ? 2 : 4, pass_lds_of(logn, tsize, true));
}

constexpr int col_blocks_per_cu(int logn, int tsize) {
  return lds_blocks(logn >= 7 ? 2 : 4, pass_lds_of(logn, tsize, false));
}
static_assert(dst_blocks_per_cu(9, 8) == 2 && dst_blocks_per_cu(10, 8) == 1 && dst_blocks_per_cu(11, 8) == 2 &&
                  dst_blocks_per_cu(10, 4) == 2 && col_blocks_per_cu(10, 8) == 1 && col_blocks_per_cu(11, 8) == 2,
              "workgroups of long rows per CU");

// Calls f(e) for e = t + u kBlock, u = 0 .. TOTAL / kBlock - 1 (TOTAL a
// multiple of kBlock known at compile time), fully unrolled: with the row
// length a compile-time power of two, the row and column of e and their LDS
// offsets fold to per-thread constants plus immediates.
template <int TOTAL, typename F>
__device__ __forceinline__ void for_elems_ct(F&& f) {
  static_assert(TOTAL % kBlock == 0, "whole multiples of the workgroup");
  const int t = static_cast<int>(threadIdx.x) & (kBlock - 1);
#pragma unroll
  for (int u = 0; u < TOTAL / kBlock; ++u) f(t + u * kBlock);
}

// The elements of a block of RC rows of n = 2^LOGN.
template <int RC, int LOGN, typename F>
__device__ __forceinline__ void for_row_elems(F&& f) {
  for_elems_ct<(RC << LOGN)>(f);
}

// The elements of a block of rows in batches of up to U: load(e, v) for every
// element of a batch, then V::pin, then use(u, e, v) (u = e / kBlock).  Every
// load of a batch is in flight before the first use.
template <int B, typename V, typename L, typename S>
__device__ __forceinline__ void elem_batch(int it, L& load, S& use) {
  V v[B];
#pragma unroll
  for (int u = 0; u < B; ++u) load(static_cast<int>(threadIdx.x) + (it + u) * kBlock, v[u]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < B; ++u) v[u].pin();
#pragma unroll
  for (int u = 0; u < B; ++u) use(it + u, static_cast<int>(threadIdx.x) + (it + u) * kBlock, v[u]);
}
template <int RC, int LOGN, int U, typename V, typename L, typename S>
__device__ __forceinline__ void for_row_batches(L&& load, S&& use) {
  constexpr int NIT = (RC << LOGN) / kBlock;
  constexpr int B = NIT < U ? NIT : U;
  static_assert(NIT >= 1 && NIT % B == 0, "whole batches");
#pragma unroll
  for (int it = 0; it < NIT; it += B) elem_batch<B, V>(it, load, use);
}

// Elements per batch of a source assembly with five to seven loads each:
// what the register budget of the pass holds in flight.
template <typename T, int LOGN>
constexpr int src_batch() {
  return sizeof(T) == 4 && sym_core(4, 1 << LOGN) && (1 << LOGN) >= 256 ? 8 : 4;
}

// Element e of a block of R = 2^lr rows in the strip order (Geom::strip): e =
// 4 R s + 4 r + c is row r, column 4 s + c, stored at offset (s ny + j0 + r) 4
// + c of the plane, so 4 R consecutive elements are one block in memory.
__device__ __forceinline__ void strip_elem(int e, int lr, int& r, int& i) {
  const int w = e & ((4 << lr) - 1);
  r = w >> 2;
  i = ((e >> (lr + 2)) << 2) | (w & 3);
}
__device__ __forceinline__ unsigned int strip_off(int e, int lr, int j0, int ny) {
  return static_cast<unsigned int>(e >> (lr + 2)) * (static_cast<unsigned int>(ny) << 2) +
         (static_cast<unsigned int>(j0) << 2) + (e & ((4 << lr) - 1));
}
__host__ __device__ constexpr int log2_rows(int R) {
  int l = 0;
  while ((1 << l) < R) ++l;
  return l;
}

// The RC rows j0.. of a row block between LDS and an intermediate plane of a
// solve: row-major, or in the strip order (Geom::strip).
template <typename T, int RC, int LOGN>
__device__ __forceinline__ void rows_to_plane(const Geom& g, int j0, const T* buf, int ppitch,
                                              T* __restrict__ out) {
  constexpr int n = 1 << LOGN;
  if (g.strip) {
    for_row_elems<RC, LOGN>([&](int e) {
      int r, i;
      strip_elem(e, log2_rows(RC), r, i);
      store_at(out, strip_off(e, log2_rows(RC), j0, g.ny), buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)]);
    });
  } else {
    for_row_elems<RC, LOGN>([&](int e) {
      const int r = e >> LOGN, i = e & (n - 1);
      store_at(out, (j0 + r) * n + i, buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)]);
    });
  }
}
// The way back in two halves: all loads, then (after whatever other
// loads the pass has) the LDS stores.
template <typename T, int RC, int LOGN>
struct RowFetch {
  static constexpr int N = (RC << LOGN) / kBlock;
  T v[N];
  // (one branch on the plane order around all of them: a select per address
  // becomes a branch per load)
  __device__ __forceinline__ void load(const Geom& g, int j0, const T* __restrict__ in) {
    const unsigned int t = threadIdx.x;
    if (g.strip) {
#pragma unroll
      for (int u = 0; u < N; ++u)
        v[u] = load_at(in, strip_off(t + u * kBlock, log2_rows(RC), j0, g.ny));
    } else {
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = load_at(in, (static_cast<unsigned int>(j0) << LOGN) + t + u * kBlock);
    }
  }
  __device__ __forceinline__ void put(const Geom& g, T* buf, int ppitch) {
    constexpr int n = 1 << LOGN;
    const int t = static_cast<int>(threadIdx.x);
#pragma unroll
    for (int u = 0; u < N; ++u) pin(v[u]);
    if (g.strip) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        int r, i;
        strip_elem(t + u * kBlock, log2_rows(RC), r, i);
        buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)] = v[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int e = t + u * kBlock;
        buf[RowLay<T, LOGN>::rpos(n, ppitch, e >> LOGN, e & (n - 1))] = v[u];
      }
    }
  }
};

// Source assembly (FP64) of the rows j0.. of the Bx/By predictor-corrector:
//   FX:      -d_y Jz + (Jy_{k-1} - Jy_{k+1}) / (2 dzeta) - shift * Bx_old
//   else:     d_x Jz - (Jx_{k-1} - Jx_{k+1}) / (2 dzeta) - shift * By_old
template <typename T, int LOGN, bool FX>
__device__ __forceinline__ void src_bxby_rows(const Geom& g, const SrcBxBy<T>& a, int j0, T* buf,
                                              int ppitch) {
  constexpr int n = 1 << LOGN, R = pass_rows<T>(n);
  const double ih = FX ? -0.5 / g.hy : 0.5 / g.hx;
  const double idz = FX ? 0.5 / a.dzeta : -0.5 / a.dzeta;
  const double amp = a.beam_amp;
  const double* __restrict__ jz = a.jz;
  const double* __restrict__ prev = FX ? a.jy_prev : a.jx_prev;
  const double* __restrict__ next = FX ? a.jy_next : a.jx_next;
  const double* __restrict__ shrd = FX ? a.sy_next : a.sx_next;
  const T* __restrict__ bold = FX ? a.bx : a.by;
  // Gaussian profile factors: along x those of the thread's columns i = t +
  // 256 c, along y those of the block's rows where a row is whole workgroups
  // wide (uniform), else per element
  constexpr int NC = n > kBlock ? n / kBlock : 1;
  constexpr bool rows_uniform = n >= kBlock;
  double gx0[NC], gx1[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int i = (static_cast<int>(threadIdx.x) + c * kBlock) & (n - 1);
    gx0[c] = load_at(a.bgx, FX ? i : (i > 0 ? i - 1 : 0));
    gx1[c] = FX ? gx0[c] : load_at(a.bgx, i + 1);
  }
  double gy[rows_uniform ? R + 2 : 1];
  if constexpr (rows_uniform) {
#pragma unroll
    for (int q = 0; q < R + 2; ++q) gy[q] = a.bgy[j0 + q > 0 ? j0 + q - 1 : 0];
  }
  struct In {
    double z0, z1, p, t, s, g0, g1;
    T b;
    __device__ void pin() {
      dst_detail::pin(z0);
      dst_detail::pin(z1);
      dst_detail::pin(p);
      dst_detail::pin(t);
      dst_detail::pin(s);
      dst_detail::pin(b);
      if constexpr (!rows_uniform) {
        dst_detail::pin(g0);
        dst_detail::pin(g1);
      }
    }
  };
  for_row_batches<R, LOGN, src_batch<T, LOGN>(), In>(
      [&](int e, In& v) {
        const int i = e & (n - 1), j = j0 + (e >> LOGN);
        const int o = j * n + i;
        // neighbours with clamped indices, replaced by selects below
        v.z0 = load_at(jz, FX ? (j > 0 ? o - n : o) : (i > 0 ? o - 1 : o));
        v.z1 = load_at(jz, FX ? (j + 1 < g.ny ? o + n : o) : (i + 1 < n ? o + 1 : o));
        v.p = load_at(prev, o);
        v.t = load_at(next, o);
        v.s = load_at(shrd, o);
        v.b = load_at(bold, o);
        if constexpr (!rows_uniform) {
          v.g0 = load_at(a.bgy, FX ? (j > 0 ? j - 1 : 0) : j);
          v.g1 = load_at(a.bgy, FX ? j + 1 : j);
        }
      },
      [&](int u, int e, const In& v) {
        const int r = e >> LOGN, i = e & (n - 1), j = j0 + r;
        const int c = u % NC;
        double g0 = v.g0, g1 = v.g1;
        if constexpr (rows_uniform) {
          g0 = gy[FX ? u / NC : u / NC + 1];
          g1 = gy[FX ? u / NC + 2 : u / NC + 1];
        }
        const double q0 = v.z0 - amp * gx0[c] * g0;
        const double q1 = (FX ? j + 1 < g.ny : i + 1 < n) ? v.z1 - amp * gx1[c] * g1 : 0.0;
        const double q = (q1 - q0) * ih + (v.p - (v.t + v.s)) * idz - a.shift * static_cast<double>(v.b);
        buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)] = static_cast<T>((i > 0 && j > 0) ? q : 0.0);
      });
}

// Source assembly (FP64) + forward DST along x of row block bxi of field
// fld (0 Bx, 1 By) of the Bx/By predictor-corrector.
template <typename T, int LOGN>
__device__ __forceinline__ void src_bxby_block(const Geom& g, const SrcBxBy<T>& a,
                                               const AxisTables<T>& tx, int bxi, int fld,
                                               unsigned char* smem_raw) {
  __syncthreads();   // the workgroup's previous use of LDS is complete
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  const int j0 = bxi * R;
  if (fld == 0)
    src_bxby_rows<T, LOGN, true>(g, a, j0, buf, ppitch);
  else
    src_bxby_rows<T, LOGN, false>(g, a, j0, buf, ppitch);
  xf.commit();
  __syncthreads();
  block_dst<T, LOGN, true>(buf, ppitch, xf);
  rows_to_plane<T, R, LOGN>(g, j0, buf, ppitch, a.out + static_cast<size_t>(fld) * g.nx * g.ny);
}

// Calls f(it) for it = 0 .. NIT-1 in unrolled chunks of up to 32 (NIT a
// compile-time count), so that element addresses are affine in it.
template <int NIT, typename F>
__device__ __forceinline__ void for_iters(F&& f) {
#pragma unroll
  for (int i0 = 0; i0 < NIT; i0 += 32) {
#pragma unroll
    for (int u = 0; u < (NIT - i0 < 32 ? NIT - i0 : 32); ++u) f(i0 + u);
  }
}

// Column pass with one of the FFT cores (W = 2 or 4 columns): strip load,
// forward core whose output stage divides by the eigenvalues, inverse core,
// store.  Strip-ordered planes (W = 4): the strip is one contiguous block, 4
// consecutive values per row and thread.  Row-major planes: thread t handles
// column c = t mod W and rows j = t / W + it (256 / W); the row step is a
// multiple of the LDS layout's run, so the padded index of a thread's rows is
// affine in it.
template <typename T, int LOGN, int W>
__device__ __forceinline__ void col_block_core(const Geom& g, const ColArgs<T>& a,
                                               const AxisTables<T>& ty,
                                               const double* __restrict__ lamx, int strip, int fld,
                                               unsigned char* smem_raw) {
  using Pd = CoreLay<T>;
  constexpr int n = 1 << LOGN;
  constexpr bool sym = sym_core(sizeof(T), n);
  constexpr bool once = eigen_once<T, n>;     // the eigenvalue of each slot from two of them
  constexpr int NK = sym ? 16 : n / 64;       // output slots per lane
  constexpr int LW = W == 2 ? 1 : 2;
  constexpr int JS = kBlock / W;              // row step of a thread
  constexpr int NIT = n / JS;                 // rows per thread
  constexpr int LS = Pd::ridx(JS);            // LDS step of ridx
  constexpr int rl = Pd::rlen(n);
  static_assert((W == 2 || W == 4) && n >= JS, "whole steps of rows");
  static_assert(JS % (1 << Pd::S) == 0, "row step must keep the LDS padding affine");
  T* buf = reinterpret_cast<T*>(smem_raw);
  const int nx = g.nx;
  constexpr int ppitch = pair_pitch<T>(n);
  const int p0 = strip * W;
  const int tid = static_cast<int>(threadIdx.x);
  const Xform<T, LOGN, W / 2> xf =
      stage_tables<T, LOGN, W / 2>(ty, smem_raw + static_cast<size_t>(W / 2) * ppitch * sizeof(T));
  // the y eigenvalues of the lane's core outputs, fetched under the strip
  // load: by the lane itself (wave core), or through the exchange region of
  // the first pair (symmetric core: 16 scattered values a lane)
  double ly[NK];
  double lxa = 0.0, lxb = 0.0;
  bool busy;
  int pr;                                     // pair whose outputs the lane scales
  constexpr int NLAM = n >= kBlock ? n / kBlock : 1;
  double lam_v[NLAM];
  double* lam_s = nullptr;
  if constexpr (sym) {
    const SymLane<LOGN, W / 2> t;
    pr = t.pair_b;
    busy = t.row;
    if constexpr (once) {
      // k0 of slot 0 (EigenOnce)
      static_assert(Sym<LOGN>::G == 16 && n == 2048, "outputs k0 + 256 q");
      const int k0 = t.k1 + 16 * t.g;
      lam_v[0] = ty.lam[k0];
      lam_v[1] = ty.lam[k0 + n / 2];
    } else {
      lam_s = reinterpret_cast<double*>(buf + Sym<LOGN>::template soff<T>());
      static_assert(sizeof(double) * n <= sizeof(Cplx<T>) * 9 * Sym<LOGN>::RP, "eigenvalues fit the exchange region");
#pragma unroll
      for (int u = 0; u < NLAM; ++u) lam_v[u] = ty.lam[n >= kBlock ? tid + u * kBlock : tid & (n - 1)];
    }
  } else {
    pr = tid >> 6;
    busy = pr < W / 2;
    if (busy) {
#pragma unroll
      for (int q = 0; q < NK; ++q) ly[q] = ty.lam[core_out_k<n / 32>(tid & 63, q)];
    }
  }
  lxa = lamx[p0 + (busy ? 2 * pr : 0)];
  lxb = lamx[p0 + (busy ? 2 * pr + 1 : 1)];
  bool hold = false;
  if constexpr (sizeof(T) == 8) hold = eigen_range(g, a.shift[fld], 0.25 * static_cast<double>(nx) * n);
  const size_t plane = static_cast<size_t>(nx) * n;
  const int c = tid & (W - 1), j0 = tid >> LW;
  const int lcol = (c >> 1) * ppitch + (c & 1) * rl + Pd::ridx(j0);
  const bool cont = W == 4 && g.strip != 0;
  constexpr int NQ = n >= kBlock ? n / kBlock : 1;
  struct alignas(16) Vec {
    T v[4];
  };
  if (cont) {
    const Vec* src = reinterpret_cast<const Vec*>(a.in + fld * plane + static_cast<size_t>(strip) * 4 * n);
    Vec v[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u)
      if (n >= kBlock || tid < n) v[u] = src[tid + u * kBlock];
#pragma unroll
    for (int u = 0; u < NQ; ++u)
      if (n >= kBlock || tid < n) {
        T* d = buf + Pd::ridx(tid) + Pd::ridx(u * kBlock);
        d[0] = v[u].v[0];
        d[rl] = v[u].v[1];
        d[ppitch] = v[u].v[2];
        d[ppitch + rl] = v[u].v[3];
      }
  } else {
    const T* in = a.in + fld * plane + p0 + c + static_cast<size_t>(j0) * nx;
    T* d = buf + lcol;
    for_iters<NIT>([&](int it) { d[it * LS] = in[static_cast<size_t>(it) * JS * nx]; });
  }
  xf.commit();
  if constexpr (sym && !once) {
#pragma unroll
    for (int u = 0; u < NLAM; ++u)
      if (n >= kBlock || tid < n) lam_s[tid + u * kBlock] = lam_v[u];
  }
  __syncthreads();
  {
    if constexpr (sym && !once) {
      const SymLane<LOGN, W / 2> t;
      if (busy) {
#pragma unroll
        for (int q = 0; q < NK; ++q) {
          bool stored;
          const int k = sym_out_k(t, q, stored);
          ly[q] = lam_s[stored ? k : 1];      // an unstored slot divides by something finite
        }
      }
    }
    const double shift = a.shift[fld];
    const double inorm = 0.25 * static_cast<double>(nx) * n;
    std::conditional_t<once, EigenOnce, EigenScale<T, NK>> sc;
    if (busy) {
      if constexpr (once) {
        const double two = 2.0 / (g.hy * g.hy);
        sc.c = (lam_v[0] + two) * inorm;
        sc.s = (lam_v[1] + two) * inorm;
        sc.xa = (lxa - shift - two) * inorm;
        sc.xb = (lxb - shift - two) * inorm;
      } else {
#pragma unroll
        for (int q = 0; q < NK; ++q) sc.ry[q] = static_cast<T>((ly[q] - shift) * inorm);
        sc.xa = static_cast<T>(lxa * inorm);
        sc.xb = static_cast<T>(lxb * inorm);
      }
      if constexpr (sizeof(T) == 8) {
        if (hold) {
#pragma unroll
          for (int q = 0; q < NK; ++q) sc.ry[q] = fmax(sc.ry[q], -0x1p1022);
          sc.xa = fmax(sc.xa, -0x1p1022);
          sc.xb = fmax(sc.xb, -0x1p1022);
        }
      }
      sc.za = p0 + 2 * pr == 0;
    }
    if constexpr (sym) {
      // the side job's stores drain under the transforms (which issue no
      // global loads here: a wait on a load also waits on earlier stores)
      zero_job(a.zero, static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x,
               static_cast<size_t>(gridDim.x) * gridDim.y);
      if constexpr (!once) __syncthreads();   // the eigenvalues have left the exchange region
      sym_dst<T, double, double, LOGN, W / 2>(buf, xf.w, xf.tw(), sc);
      __syncthreads();   // the rows are the next transform's input
      sym_dst<T, T, T, LOGN, W / 2>(buf, xf.w, xf.tw());
    } else if (busy) {
      float* g2 = buf + static_cast<size_t>(pr) * ppitch;
      wave_dst_core<n / 32>(g2, xf.w.a, xf.tw(), sc);
      wave_dst_core<n / 32>(g2, xf.w.a, xf.tw());
    }
  }
  __syncthreads();
  const T mihy = static_cast<T>(-0.5 / g.hy);
  const bool with_dy = fld == 0 && a.out_dy;
  if (cont) {
    const size_t sb = static_cast<size_t>(strip) * 4 * n;
    Vec* dst = reinterpret_cast<Vec*>(a.out + fld * plane + sb);
    Vec* dy = with_dy ? reinterpret_cast<Vec*>(a.out_dy + sb) : nullptr;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int j = tid + u * kBlock;
      if (n < kBlock && j >= n) break;
      const T* q = buf + Pd::ridx(j);
      dst[j] = Vec{{q[0], q[rl], q[ppitch], q[ppitch + rl]}};
      if (dy) {
        // -d_y by central differences, zero on row 0 and beyond row n - 1
        // (neighbour indices clamped into the strip)
        const T* qu = buf + Pd::ridx(j + 1 < n ? j + 1 : j);
        const T* qd = buf + Pd::ridx(j > 0 ? j - 1 : 0);
        const bool hu = j + 1 < n, in = j > 0;
        Vec d4;
        constexpr int off[4] = {0, rl, ppitch, ppitch + rl};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          d4.v[e] = in ? mihy * ((hu ? qu[off[e]] : T(0)) - qd[off[e]]) : T(0);
        dy[j] = d4;
      }
    }
    return;
  }
  T* out = a.out + fld * plane + p0 + c + static_cast<size_t>(j0) * nx;
  const T* r = buf + lcol;
  if (with_dy) {
    // -d_y by central differences, zero on the boundary rows j = 0 and the
    // clamped neighbour beyond j = ny - 1; j + 1 (j - 1) crosses a padding
    // gap exactly when j0 + 1 (j0) is a multiple of the layout's run
    T* dy = a.out_dy + p0 + c + static_cast<size_t>(j0) * nx;
    const int up = Pd::ridx(j0 + 1) - Pd::ridx(j0), dn = Pd::ridx(j0 - 1) - Pd::ridx(j0);
    for_iters<NIT>([&](int it) {
      const T* q = r + it * LS;
      const int j = j0 + it * JS;
      // the neighbour reads stay inside the strip (clamped at the two ends)
      const T v = q[0];
      const T vu = j + 1 < n ? q[j == n - 1 ? 0 : up] : T(0);
      const T vd = j > 0 ? q[j == 0 ? 0 : dn] : T(0);
      out[static_cast<size_t>(it) * JS * nx] = v;
      dy[static_cast<size_t>(it) * JS * nx] = j > 0 ? mihy * (vu - vd) : T(0);
    });
  } else {
    for_iters<NIT>([&](int it) { out[static_cast<size_t>(it) * JS * nx] = r[it * LS]; });
  }
}

// The same with the matrix core: kDenseRows columns per workgroup, the
// eigenvalue division on the product's result registers.
template <typename T, int LOGN>
__device__ __forceinline__ void col_block_dense(const Geom& g, const ColArgs<T>& a, const AxisTables<T>& ty,
                                                const double* __restrict__ lamx, int strip, int fld,
                                                unsigned char* smem_raw) {
  using D = Dense<T, LOGN>;
  constexpr int n = D::n, W = kDenseRows, N = W * n / kBlock;
  T* buf = reinterpret_cast<T*>(smem_raw);
  const auto xf = stage_tables<T, LOGN, W / 2>(ty, smem_raw);
  const int p0 = strip * W;
  const int tid = static_cast<int>(threadIdx.x), wave = tid >> 6, lane = tid & 63;
  const unsigned int nx = g.nx;
  const size_t plane = static_cast<size_t>(nx) * n;
  const T* in = a.in + fld * plane;
  // element u of a thread: column c, row j0 + u kBlock / W
  const int c = tid & (W - 1), j0 = tid / W;
  constexpr int JS = kBlock / W;
  T v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) v[u] = load_at(in, (j0 + u * JS) * nx + p0 + c);
  double lx[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) lx[r] = lamx[p0 + D::template row_of<true>(lane, r)];
  double ly[D::TW];
#pragma unroll
  for (int q = 0; q < D::TW; ++q) ly[q] = ty.lam[wave < D::NW ? dense_out(n, wave * D::TW + q, lane & 15) : 0];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < N; ++u) buf[c * D::pitch + D::ridx(j0 + u * JS)] = v[u];
  __syncthreads();
  // 1 / normalisation (nx ny / 4, exact): the eigenvalue sum in FP64, the one
  // division in the field precision
  const double inorm = 0.25 * static_cast<double>(nx) * n;
  const double shift = a.shift[fld];
  T den[4 * D::TW];
#pragma unroll
  for (int q = 0; q < D::TW; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) den[4 * q + r] = static_cast<T>((lx[r] + (ly[q] - shift)) * inorm);
  dense_dst<true, T, LOGN>(buf, xf.w, [&](int q, int row, int o, T s) {
    const T z = s / den[q];
    return p0 + row > 0 && o > 0 ? z : T(0);
  });
  __syncthreads();
  dense_dst<false, T, LOGN>(buf, xf.w, [](int, int, int o, T s) { return o > 0 ? s : T(0); });
  __syncthreads();
  T* out = a.out + fld * plane;
  const T* row = buf + c * D::pitch;
#pragma unroll
  for (int u = 0; u < N; ++u) store_at(out, (j0 + u * JS) * nx + p0 + c, row[D::ridx(j0 + u * JS)]);
  if (fld == 0 && a.out_dy) {
    const T mihy = static_cast<T>(-0.5 / g.hy);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int j = j0 + u * JS;
      const T up = row[D::ridx(j + 1 < n ? j + 1 : j)], dn = row[D::ridx(j > 0 ? j - 1 : 0)];
      const T d = mihy * ((j + 1 < n ? up : T(0)) - dn);
      store_at(a.out_dy, j * nx + p0 + c, j > 0 ? d : T(0));
    }
  }
}

// DST along y, eigenvalue division, inverse DST along y (and -d_y for
// field 0 when requested) of column strip `strip` of field fld.
template <typename T, int LOGN>
__device__ __forceinline__ void col_block(const Geom& g, const ColArgs<T>& a,
                                          const AxisTables<T>& ty, const double* __restrict__ lamx,
                                          int strip, int fld, unsigned char* smem_raw) {
  constexpr int n = 1 << LOGN, W = pass_cols<T>(n);   // the launcher checks the width
  if constexpr (sym_core(sizeof(T), n) || wave_core(sizeof(T), n))
    col_block_core<T, LOGN, W>(g, a, ty, lamx, strip, fld, smem_raw);
  else
    col_block_dense<T, LOGN>(g, a, ty, lamx, strip, fld, smem_raw);
}

// Predictor-corrector epilogue: B_new from the inverse transform, FP64 sums
// of |B_new - B_old|^2 and |B_new|^2, B_old overwritten by B_new in place.
// Each workgroup leaves its two sums in a.partial; the next trial push (or
// the real push after the last iteration) forms the relative change and
// decides convergence.
template <typename T, int LOGN>
__device__ __forceinline__ void row_inv_pc_block(const Geom& g, const PCArgs<T>& a,
                                                 const AxisTables<T>& tx, int bxi, int fld,
                                                 unsigned char* smem_raw) {
  __syncthreads();   // the workgroup's previous use of LDS is complete
  T* buf = reinterpret_cast<T*>(smem_raw);
  constexpr int n = 1 << LOGN;   // = nx
  constexpr int R = pass_rows<T>(n);
  constexpr int ppitch = pair_pitch<T>(n);
  const auto xf = stage_row_tables<T, LOGN>(tx, smem_raw);
  const int j0 = bxi * R;
  T* b = fld == 0 ? a.bx : a.by;
  T* tp = fld == 0 ? a.tape_bx : a.tape_by;
  const T* in = a.in + static_cast<size_t>(fld) * g.nx * g.ny;
  // the old iterate is fetched under the plane load (its own round trip after
  // the transform took 2.8k of 18.4k cycles at 1024^2 in FP32)
  constexpr int NOLD = (R << LOGN) / kBlock;
  T old_b[NOLD];
  RowFetch<T, R, LOGN> rows;
  rows.load(g, j0, in);
#pragma unroll
  for (int u = 0; u < NOLD; ++u) old_b[u] = load_at(b, j0 * n + static_cast<int>(threadIdx.x) + u * kBlock);
  __builtin_amdgcn_sched_barrier(0);
  rows.put(g, buf, ppitch);
#pragma unroll
  for (int u = 0; u < NOLD; ++u) pin(old_b[u]);
  xf.commit();
  __syncthreads();
  block_dst<T, LOGN, false>(buf, ppitch, xf);
  double dsum = 0.0, nsum = 0.0;
  auto update = [&](int e, T prev, auto taped) {
    const int r = e >> LOGN, i = e & (n - 1);
    const int j = j0 + r;
    const T v = buf[RowLay<T, LOGN>::rpos(n, ppitch, r, i)];
    const T u = j > 0 ? v : T(0);
    const double d = static_cast<double>(u) - static_cast<double>(prev);
    dsum += d * d;
    nsum += static_cast<double>(u) * static_cast<double>(u);
    store_at(b, j * n + i, u);
    if constexpr (decltype(taped)::value) store_at(tp, j * n + i, u);
  };
  auto finish = [&](auto taped) {   // the tape tested once, not per element
#pragma unroll
    for (int u = 0; u < NOLD; ++u) update(static_cast<int>(threadIdx.x) + u * kBlock, old_b[u], taped);
  };
  if (tp)
    finish(std::true_type{});
  else
    finish(std::false_type{});
  double v[2] = {dsum, nsum};
  partials::store<2>(v, a.partial, fld * (g.ny / R) + bxi);
}

}  // namespace dst_detail

}  // namespace qsp
