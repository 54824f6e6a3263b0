// Device side of the factored extrinsic likelihood for gfx950.
//
// One lane evaluates one extrinsic sample.  Per sample (Eq. (def:lnL:Decomposed)):
//   sky frame and arrival times in FP64 (the delay feeds a sub-sample read),
//   antenna factors F_k = F+ + i Fx from the shared polarisation tensors,
//   -2Y_lm(incl, phiref) from per-mode Fourier coefficients in incl,
//   the data term x Re sum conj(F_k Y) Q_k(t_k) with a four-point Lagrange read
//   of the time-major table Q[k][t][mode] (taps outside the window read 0),
//   the model-norm term x^2/4 sum_k [|F_k|^2 a_k + Re(F_k^2 b_k)].
//
// Model-norm term.  a_k = Y^H U_k Y and b_k = Y^T V_k Y depend on the sample
// only through (incl, phiref), and both are finite trigonometric polynomials:
// d^l_{m,2}(incl) has degree l in incl (even/odd in incl for even/odd m), and
// the phiref dependence of a pair of modes is e^{i(m'-m) phi} (a_k) or
// e^{i(m+m') phi} (b_k).  So with L = max l,
//   g_c(incl, phi) in { a_k/4, Re b_k/4, -Im b_k/4 }
//   = sum_b C[b][c] beta_b(incl, phi),
//   beta_b in { cos(n incl) [1 | cos(q phi) | sin(q phi)], q even,
//               sin(n incl) [cos(q phi) | sin(q phi)],     q odd },
// n <= 2L, q <= 2L, and the per-sample work is one contraction of the basis
// values with the uniform coefficient table C (scalar loads).  C is exact up
// to rounding: a setup kernel takes the phi dependence of every pair of modes as it
// stands and projects that in incl on a grid finer than twice the degree
// (discrete orthogonality).  The finite angular harmonic
// content this relies on is the paper's Eq. (ap:angleharm) argument applied to
// (incl, phiref).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace rift {

constexpr int KMAX = 8;    // detectors
constexpr int MMAX = 25;   // modes
constexpr int LMAXC = 8;   // largest l
constexpr int QPAD = 4;    // zero rows on each side of every Q series
// Q tables hold W consecutive (internal) modes per time row.  FP64: W = 8, a row
// of a group one aligned 128-byte line, where q_width64 says so; otherwise W = 2,
// whose four stencil rows of a group are 128 bytes at any multiple of 32.  FP32: W = 4,
// 32-byte rows.
constexpr int QW64 = 8;
constexpr int QW64_SHORT = 2;
constexpr int QW64_SHORT_MODES = 12;
constexpr int QW32 = 4;
__host__ __device__ constexpr int q_groups(int M, int W) { return (M + W - 1) / W; }
// The width of a point's FP64 rows, of M modes and K detectors in class L, KT the
// plan's detector class.  Per detector the reads are 4 units of 128 bytes per eight modes against
// one per two: 12 against 11 at 21 modes, where every line is used whole (12 lines
// against 19) and the contraction runs between the units.  Measured, rows of eight
// against rows of two (lnL and ln Z of 3e5 samples; the tile form of the time rules,
// 6e4 x 11 times, which the units bound; in brackets the class l <= 8):
//   KT 2:  13 modes 0.90, 0.72; 17 0.91, 0.78; 21 0.82, 0.67; (25 0.50, 0.79); two
//          detectors 21 0.94; 17 tile form 1.11, recompute of a mixed plan 1.14
//   KT 3:  13 0.99, 1.11; 14 0.98, 1.11; 15 0.93, 1.02; 16 0.97, 1.02; 17 1.06, 1.28;
//          18 1.08, 1.28; 20 0.98, 1.18; 21 0.93, 1.09; (22 0.86, 1.03; 25 0.95, 1.15;
//          their small batches 0.68)
//   KT 5:  13 1.01, 1.03; 16 0.91, 0.92; 17 1.20, 1.17; 18 1.31, 1.23; 20 1.12, 1.08;
//          21 1.01, 0.99 (small batches 0.92, 0.89); (22 1.09, 0.97; 25 1.13, 1.03)
//   KT 8:  13 1.00, 1.02; 16 0.95, 0.93; 17 1.06, 1.15; 20 1.02, 1.06; 21 0.98, 0.99;
//          (25 0.94, 0.94)
// Up to 12 modes rows of two: 9 modes, KT 3, 5e5 samples 111 us against 95.  A mixed
// plan, whose recompute alone reads the table (rows of eight 1.05 - 1.07 at 15 to 21
// modes, KT 3), takes the same rows: its recomputed samples are the FP64 plan's
// values bit for bit.
__host__ __device__ constexpr int q_width64(int M, int K, int L, int KT) {
  if (M <= QW64_SHORT_MODES) return QW64_SHORT;
  const int empty = q_groups(M, QW64) * QW64 - M;
  bool eight = empty <= 3;                                             // 13 - 16, 21 - 24
  if (KT == 2) eight = K == 1 || L == 8 || empty <= 5;
  else if (KT == 3) eight = L == 8 || M > 20 || (M > 14 && eight);
  else if (KT == 8) eight = eight || (L == 8 && M > 24);
  return eight ? QW64 : QW64_SHORT;
}
// LDS staging of the data term: one unit is the 128-byte stencil block of a
// (mode group, detector) pair for each of the 64 lanes of a wavefront; every
// wavefront owns two unit buffers.
constexpr int STAGE_UNIT = 64 * 128;
constexpr int STAGE_WAVE = 2 * STAGE_UNIT;

template <class R>
struct alignas(2 * sizeof(R)) C2 {
  R x, y;
};

// Per-point description, resident in device memory (uniform per block).
struct PointDesc {
  int32_t K;        // real detectors
  int32_t M;        // modes
  int32_t n_t;      // table samples per detector and mode
  int32_t L;        // mode class: max l rounded to 2, 3, 4 or 8
  int32_t B;        // basis functions of the class
  int32_t KT;       // detector class (padded K)
  int32_t m_min;    // smallest m (modes are stored sorted by m)
  int32_t w64;      // modes per row of the FP64 table (q_width64)
  int64_t n;        // samples of this point in a batch
  int64_t s0;       // first sample column of this point in a batch
  double t0, inv_dt, gmst, d_ref;
  double T;         // mixed path: refinement margin (nats)
  double lnN;       // ln(n)
  double dten[KMAX][6];   // D00, D11, D22, 2 D01, 2 D02, 2 D12
  double rpos[KMAX][3];   // light-seconds
  int32_t m[MMAX];        // m of internal mode i (sorted ascending)
  int32_t odd[MMAX];      // m odd
  double ycoef[MMAX][LMAXC + 1];  // d^l_{m,2}(incl) sqrt((2l+1)/4pi) = sum_n ycoef cos|sin(n incl)
  float ycoef32[MMAX][LMAXC + 1];
  float dten32[KMAX][6];
  // mixed path, a-priori bound on |lnL_FP32 - lnL_FP64| of one sample:
  //   x bnd_d + x^2 sum_k [ (|F_k| + eF[k])^2 bnd_q[k]
  //                         + (2 (|F_k| + eF[k]) eF[k] + eF[k]^2) l1q[k] ]
  // (written on the device by k_bound; see there for the derivation)
  double bnd_d;
  double bnd_q[KMAX];
  double l1q[KMAX];  // sum of |C| over detector k's three coefficient columns
  double eF[KMAX];   // bound on |F_FP32 - F| of detector k
  // arrival-time binning (sorted evaluation): a Morton key of bin_bits
  // bits per detector over the first bin_dims detectors; its top bin_cb
  // bits are the coarse bucket.  The point's sort tiles are bin_st0 ..
  // bin_st0 + bin_nst - 1; its [coarse bucket][sort tile] count matrix
  // starts at bin_mbase.
  int32_t bin_dims;
  int32_t bin_bits;
  int32_t bin_cb;
  int32_t bin_nst;
  int32_t bin_st0;
  int32_t bin_pad;
  int64_t bin_mbase;
  // Q of each detector in groups of W internal modes, QPAD zero rows at both
  // ends of every series: [KT][ceil(M / W)][n_t + 2 QPAD][W] complex, the
  // slots past M zero.  A stencil starting at row j-1 in [-QPAD, n_t] reads
  // padded rows j-1+QPAD .. j+2+QPAD.
  const double* Q64;
  const float* Q32;
  const double* C64;      // [B][3 KT]
  const float* C32;       // [B][3 KT]
};

// Work unit: samples [s, s + cnt) (global columns) of point p.
struct Tile {
  int32_t p;
  int32_t cnt;
  int64_t s;
};

template <int L>
struct Cls {
  static constexpr int NI = 2 * L;                        // incl degree of g_c
  static constexpr int NQ = 2 * L;                        // phi degree of g_c
  static constexpr int MAXM = (L == 2) ? 5 : (L == 3) ? 12 : (L == 4) ? 21 : 25;
  static constexpr int NY = L + 1;                        // Fourier terms of d_lm
  static constexpr int B = (NI + 1) + (NQ / 2) * 2 * (NI + 1) + ((NQ + 1) / 2) * 2 * NI;
};


__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Address spaces: the point description and the coefficient tables are read
// with uniform addresses through the constant space (scalar loads into
// SGPRs); per-lane data (samples, the Q table, outputs) through the global
// space (vector loads).
#define RIFT_CONST __attribute__((address_space(4)))
#define RIFT_GLOBAL __attribute__((address_space(1)))
#define RIFT_LDS __attribute__((address_space(3)))

struct PointDesc;
typedef const RIFT_CONST PointDesc* PDesc;

template <class T>
__device__ __forceinline__ const RIFT_CONST T* as_const(const T* p) {
  return (const RIFT_CONST T*)p;
}
template <class T>
__device__ __forceinline__ const RIFT_GLOBAL T* as_global(const T* p) {
  return (const RIFT_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ RIFT_GLOBAL T* as_global_w(T* p) {
  return (RIFT_GLOBAL T*)p;
}

// Identity the optimiser cannot see through.  Applied to the (uniform) point
// pointer at the top of every sample iteration so that the ~10^3 uniform
// coefficient loads of a sample stay scalar loads inside the loop instead of
// being hoisted out of it.
template <class T>
__device__ __forceinline__ const RIFT_CONST T* opaque(const T* p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (const RIFT_CONST T*)v;
}
template <class T>
__device__ __forceinline__ const RIFT_CONST T* opaque(const RIFT_CONST T* p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (const RIFT_CONST T*)v;
}
// Empty register use: the value must be computed before this point.
template <class R>
__device__ __forceinline__ void pin(R& v) {
  asm volatile("" : "+v"(v));
}
// Empty scalar use: the (uniform) value must be in SGPRs at this point.
template <class R>
__device__ __forceinline__ void pin_s(R v) {
  asm volatile("" ::"s"(v));
}
// Element k (uniform) of a per-detector value in registers.  The operands are
// opaque: a selection between plain elements turns into an indexed read, and
// puts the array into scratch.
template <int KT, class T>
__device__ __forceinline__ T by_det(const T* v, int k) {
  T r = v[0];
  pin(r);
#pragma unroll
  for (int j = 1; j < KT; ++j) {
    T t = v[j];
    pin(t);
    r = k == j ? t : r;
  }
  return r;
}
// sin and cos of N angles at once: Cody and Waite's reduction by pi/2 in three
// parts with fused multiply-adds, then the Taylor series through r^17 and r^18 on |r| <= pi/4
// (truncation below 1e-18), the N angles side by side, so that each constant is
// fetched once and the chains of one angle fill the latencies of another's:
// 36 vector operations an angle, where the library's function takes 105.
// Angles beyond 2^30 go to that.
struct SinCosTab {
  double two_over_pi, p1, p2, p3;
  double s[8], c[9];
};
__constant__ const SinCosTab kSinCos = {
    0.6366197723675814,
    1.5707963267948966,
    6.123233995736766e-17,
    -1.4973849048591698e-33,
    {-1.0 / 6.0, 1.0 / 120.0, -1.0 / 5040.0, 1.0 / 362880.0, -1.0 / 39916800.0, 1.0 / 6227020800.0,
     -1.0 / 1307674368000.0, 1.0 / 355687428096000.0},
    {-0.5, 1.0 / 24.0, -1.0 / 720.0, 1.0 / 40320.0, -1.0 / 3628800.0, 1.0 / 479001600.0, -1.0 / 87178291200.0,
     1.0 / 20922789888000.0, -1.0 / 6402373705728000.0}};
template <int N>
__device__ __forceinline__ void sincos_near(const double* x, double* s, double* c) {  // |x| <= 2^30
  const RIFT_CONST SinCosTab* T = opaque(&kSinCos);
  double r[N], z[N], ps[N], pc[N];
  int q[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const double k = rint(x[j] * T->two_over_pi);
    r[j] = fma(-k, T->p3, fma(-k, T->p2, fma(-k, T->p1, x[j])));
    q[j] = (int)k;
    z[j] = r[j] * r[j];
    ps[j] = T->s[7];
    pc[j] = T->c[8];
  }
#pragma unroll
  for (int t = 7; t >= 0; --t)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (t < 7) ps[j] = fma(ps[j], z[j], T->s[t]);
      pc[j] = fma(pc[j], z[j], T->c[t]);
    }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const double sr = fma(ps[j] * z[j], r[j], r[j]), cr = fma(pc[j], z[j], 1.0);
    const double a = (q[j] & 1) ? cr : sr, b = (q[j] & 1) ? sr : cr;
    s[j] = (q[j] & 2) ? -a : a;
    c[j] = ((q[j] + 1) & 2) ? -b : b;
  }
}
template <int N>
__device__ __forceinline__ void sincos_many(const double* x, double* s, double* c) {
  sincos_near<N>(x, s, c);
  bool far = false;
#pragma unroll
  for (int j = 0; j < N; ++j) far = far || fabs(x[j]) > 1073741824.0;
  if (__any(far)) {
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (fabs(x[j]) > 1073741824.0) sincos(x[j], &s[j], &c[j]);
  }
}
// Pin a (uniform) global pointer to SGPRs, so that per-lane accesses at a
// 32-bit offset from it use the scalar-base addressing form.
__device__ __forceinline__ const RIFT_GLOBAL char* uniform_ptr(const RIFT_GLOBAL char* p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (const RIFT_GLOBAL char*)v;
}
template <class R>
__device__ __forceinline__ C2<R> ldq(const RIFT_GLOBAL R* q, int64_t idx) {
  C2<R> v;
  v.x = q[2 * idx];
  v.y = q[2 * idx + 1];
  return v;
}

template <class R>
struct Tab;
template <>
struct Tab<double> {
  static constexpr int W = QW64_SHORT;
  static __device__ __forceinline__ const RIFT_GLOBAL double* Q(PDesc P) { return as_global(P->Q64); }
  static __device__ __forceinline__ const RIFT_CONST double* C(PDesc P) { return as_const(P->C64); }
  static __device__ __forceinline__ double y(PDesc P, int i, int n) { return P->ycoef[i][n]; }
  static __device__ __forceinline__ double d(PDesc P, int k, int a) { return P->dten[k][a]; }
};
template <>
struct Tab<float> {
  static constexpr int W = QW32;
  static __device__ __forceinline__ const RIFT_GLOBAL float* Q(PDesc P) { return as_global(P->Q32); }
  static __device__ __forceinline__ const RIFT_CONST float* C(PDesc P) { return as_const(P->C32); }
  static __device__ __forceinline__ float y(PDesc P, int i, int n) { return P->ycoef32[i][n]; }
  static __device__ __forceinline__ float d(PDesc P, int k, int a) { return P->dten32[k][a]; }
};

// Row b of the harmonic basis of class L (the order of the coefficient
// table): kind 0 = cos(n incl); 1, 2 = cos(n incl) {cos, sin}(q phi) for even
// q >= 2; 3, 4 = sin(n incl) {cos, sin}(q phi) for odd q.  Packed as
// kind | n << 4 | q << 12.
template <int L>
__host__ __device__ constexpr int basis_row(int b) {
  constexpr int NI = 2 * L;
  int bb = b;
  for (int q = 0; q <= NI; ++q) {
    if (q == 0) {
      if (bb <= NI) return 0 | (bb << 4);
      bb -= NI + 1;
    } else if ((q & 1) == 0) {
      if (bb < 2 * (NI + 1)) return (1 + (bb & 1)) | ((bb >> 1) << 4) | (q << 12);
      bb -= 2 * (NI + 1);
    } else {
      if (bb < 2 * NI) return (3 + (bb & 1)) | ((1 + (bb >> 1)) << 4) | (q << 12);
      bb -= 2 * NI;
    }
  }
  return -1;
}

// Model-norm contraction acc[c] = sum_b C[b][c] beta_b(incl, phi), fully
// unrolled over the B x 3 KT coefficients (classes L <= 4): every index is a
// template constant, so the tables below stay in registers.  The uniform
// coefficients stream through SGPRs in chunks of 128 bytes, each chunk
// prefetched while the previous one is used.  Scalar loads complete out of
// order, so the wait for a chunk (pin_s) comes before the next chunk is
// issued (a wait never covers the prefetch), and the accumulators are pinned
// after each chunk's FMAs so that those FMAs stay ahead of the next wait.
template <class R, int KT, int L>
struct Contract {
  static constexpr int NI = 2 * L;
  static constexpr int W = 3 * KT;
  static constexpr int NC = Cls<L>::B * W;
  static constexpr int CH = 128 / (int)sizeof(R);
  static constexpr int NCH = (NC + CH - 1) / CH;
  struct Tabs {
    R ct[NI + 1], st[NI + 1];  // cos(n incl), sin(n incl)
    R ex[NI + 1], ey[NI + 1];  // e^{i q phi}
  };

  template <int J>
  static __device__ __forceinline__ void coef(R c, R* acc, const Tabs& T) {
    if constexpr (J < NC) {
      constexpr int rb = basis_row<L>(J / W);
      constexpr int kind = rb & 15, n = (rb >> 4) & 255, q = rb >> 12;
      R beta;
      if constexpr (kind == 0) beta = T.ct[n];
      else if constexpr (kind == 1) beta = T.ct[n] * T.ex[q];
      else if constexpr (kind == 2) beta = T.ct[n] * T.ey[q];
      else if constexpr (kind == 3) beta = T.st[n] * T.ex[q];
      else beta = T.st[n] * T.ey[q];
      acc[J % W] = fma(c, beta, acc[J % W]);
    }
  }
  template <int C, int... I>
  static __device__ __forceinline__ void fm(const R (&buf)[CH], R* acc, const Tabs& T,
                                            std::integer_sequence<int, I...>) {
    (coef<C * CH + I>(buf[I], acc, T), ...);
  }
  template <int C>
  static __device__ __forceinline__ void ld(R (&buf)[CH], const RIFT_CONST R* Cc) {
    const RIFT_CONST R* p = opaque(Cc) + C * CH;
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (C * CH + i < NC) buf[i] = p[i];
  }
  template <int C>
  static __device__ __forceinline__ void wait(const R (&buf)[CH]) {
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (C * CH + i < NC) pin_s(buf[i]);
  }
  template <int C>
  static __device__ __forceinline__ void step(const RIFT_CONST R* Cc, R (&cur)[CH], R (&nxt)[CH],
                                              R* acc, const Tabs& T) {
    if constexpr (C < NCH) {
      wait<C>(cur);
      if constexpr (C + 1 < NCH) ld<C + 1>(nxt, Cc);
      fm<C>(cur, acc, T, std::make_integer_sequence<int, CH>{});
#pragma unroll
      for (int c = 0; c < W; ++c) pin(acc[c]);
      step<C + 1>(Cc, nxt, cur, acc, T);
    }
  }
  static __device__ __forceinline__ void run(PDesc P, R ci, R si, R cf, R sf, R* acc) {
    Tabs T;
    T.ct[0] = 1;
    T.st[0] = 0;
    T.ct[1] = ci;
    T.st[1] = si;
#pragma unroll
    for (int n = 2; n <= NI; ++n) {
      T.ct[n] = 2 * ci * T.ct[n - 1] - T.ct[n - 2];
      T.st[n] = 2 * ci * T.st[n - 1] - T.st[n - 2];
    }
    T.ex[0] = 1;
    T.ey[0] = 0;
    T.ex[1] = cf;
    T.ey[1] = sf;
#pragma unroll
    for (int q = 2; q <= NI; ++q) {
      T.ex[q] = T.ex[q - 1] * cf - T.ey[q - 1] * sf;
      T.ey[q] = T.ex[q - 1] * sf + T.ey[q - 1] * cf;
    }
    const RIFT_CONST R* Cc = Tab<R>::C(P);
    R bA[CH], bB[CH];
    ld<0>(bA, Cc);
    step<0>(Cc, bA, bB, acc, T);
  }
};

// Per-mode arithmetic of the data term, every multiply-add written as an
// explicit fma (with multiply-adds otherwise fused only within one source
// expression, an expression gives the same bits in every kernel that inlines
// it).
//   phase_up: ph <- ph e^{i phi};  phase_down: ph <- ph e^{-i phi}
template <class R>
__device__ __forceinline__ void phase_up(C2<R>& ph, R cf, R sf) {
  const R a = fma(ph.x, cf, -ph.y * sf), b = fma(ph.y, cf, ph.x * sf);
  ph.x = a;
  ph.y = b;
}
template <class R>
__device__ __forceinline__ void phase_down(C2<R>& ph, R cf, R sf) {
  const R a = fma(ph.x, cf, ph.y * sf), b = fma(ph.y, cf, -ph.x * sf);
  ph.x = a;
  ph.y = b;
}
// d_i(incl) from its Fourier coefficients (sin series for odd m).
template <class R, int NY>
__device__ __forceinline__ R mode_d(PDesc P, int i, const R* cn, const R* sn) {
  R d = 0;
  if (P->odd[i]) {
#pragma unroll
    for (int n = 1; n < NY; ++n) d = fma(Tab<R>::y(P, i, n), sn[n], d);
  } else {
#pragma unroll
    for (int n = 0; n < NY; ++n) d = fma(Tab<R>::y(P, i, n), cn[n], d);
  }
  return d;
}
// Z += conj(Y) Qhat with Qhat the Lagrange combination of four taps.
template <class R>
__device__ __forceinline__ void mode_acc(C2<R>& Z, const R* w, C2<R> q0, C2<R> q1, C2<R> q2, C2<R> q3,
                                         R yx, R yy) {
  const R qx = fma(w[3], q3.x, fma(w[2], q2.x, fma(w[1], q1.x, w[0] * q0.x)));
  const R qy = fma(w[3], q3.y, fma(w[2], q2.y, fma(w[1], q1.y, w[0] * q0.y)));
  Z.x = fma(yx, qx, Z.x);
  Z.x = fma(yy, qy, Z.x);
  Z.y = fma(yx, qy, Z.y);
  Z.y = fma(-yy, qx, Z.y);
}
// The four Lagrange weights on nodes -1, 0, 1, 2 at fraction s.
template <class R>
__device__ __forceinline__ void lagrange4(R s, R* w) {
  w[0] = -s * (s - 1) * (s - 2) * (R)(1.0 / 6.0);
  w[1] = (s + 1) * (s - 1) * (s - 2) * (R)0.5;
  w[2] = -(s + 1) * s * (s - 2) * (R)0.5;
  w[3] = (s + 1) * s * (s - 1) * (R)(1.0 / 6.0);
}

// Row coordinate of a stencil: u = (t_k - t0) / dt.  A non-finite u poisons
// the sample; a finite u far outside the stored window is moved to just
// outside it (every tap then reads a zero pad row, the zero extension of the
// window), which also keeps the integer row in range.
__device__ __forceinline__ bool stencil_u(double& u, int n_t) {
  if (!(fabs(u) <= 1.0e300)) {  // NaN or infinite
    u = 0.0;
    return false;
  }
  u = fmin(fmax(u, -2.0 * QPAD), (double)n_t + 2.0 * QPAD);
  return true;
}

// a - 2 pi rint(a / 2 pi) in FP64 (2 pi split into two doubles): the angle
// in [-pi, pi] that the FP32 arithmetic starts from, so that its rounding to
// FP32 is at most pi 2^-25 rad whatever the size of the input angle.
__device__ __forceinline__ double reduce_2pi(double a) {
  const double k = rint(a * 0.15915494309189533577);
  double r = fma(-k, 6.283185307179586232, a);
  return fma(-k, 2.4492935982947064e-16, r);
}

// Detector groups of the data term (KT >= 2): at most three detectors share
// a pass over the modes; a remainder of one is split as 2 + 2, so every group
// has two or three detectors.
__host__ __device__ constexpr int det_group_size(int KT, int j) {
  int n3 = KT / 3, r = KT % 3;
  if (r == 1) {
    n3 -= 1;
    r = 4;
  }
  if (j < n3) return 3;
  const int jj = j - n3;
  if (r == 2) return jj == 0 ? 2 : 0;
  if (r == 4) return jj < 2 ? 2 : 0;
  return 0;
}
__host__ __device__ constexpr int det_group_start(int KT, int j) {
  int s = 0;
  for (int t = 0; t < j; ++t) s += det_group_size(KT, t);
  return s;
}

// Data term of detectors K0 .. K0+G-1 (2 <= G <= 3):
//   sum_k Re[conj(F_k) sum_i conj(Y_i) Qhat_{k,i}]
//   = sum_k Fre_k Re(Z_k) + Fim_k Im(Z_k),  Z_k = sum_i conj(Y_i) Qhat_{k,i},
// with Y_i = d_i(incl) e^{i m_i phi} (modes sorted by m, so the phase walks
// upward from e^{i m_min phi}) and Qhat the four-point Lagrange read at
// fraction sfr_k of the cell that starts at byte offset boff_k.
//
// The table holds W modes per time row, so the four stencil rows of a mode
// group are one contiguous 128-byte block per lane, at a 32-bit offset from
// the uniform start of series (k, group).  The blocks are read cooperatively:
// eight lanes fetch the eight 16-byte chunks of one lane's block, so a read
// instruction touches about 8 blocks' cache lines instead of 64 (the vector
// memory path costs about one cycle per distinct line per instruction).  The
// reads go straight to LDS (global_load_lds): lane l = 8 q + c' of read t
// fetches chunk c = c' ^ key(j) of the block of lane j = 8 t + q, which lands
// at j * 128 + c' * 16 = j * 128 + (c ^ key(j)) * 16.  With key(j) =
// (j >> 1) & 7 the eight lanes of equal j * 128 mod 256 within any sixteen
// consecutive lanes read eight different 16-byte columns, so lane j's own
// reads of its chunks are free of bank conflicts.
//
// Units (group p, detector g) are streamed with g fastest through the
// wavefront's two LDS buffers: unit u+1 is in flight while unit u is
// combined.  Requires the whole wavefront to be active.
//
// With CPLX, the imaginary part Im sum_k conj(F_k) Z_k is added to *acc_im as
// well (the complex data term whose real part is returned).
template <class R, int NY, int K0, int G, bool CPLX = false>
__device__ __forceinline__ double data_group(PDesc P, const RIFT_GLOBAL char* Qb, uint64_t gstride,
                                             uint64_t kstride, int M, int NGR, const uint32_t* boff,
                                             RIFT_LDS unsigned char* stage, const R* sfr, const R* Fre,
                                             const R* Fim, const R* cn, const R* sn, R cf, R sf,
                                             double* acc_im = nullptr) {
  static_assert(G >= 2 && G <= 3, "detector groups of two or three");
  constexpr int W = Tab<R>::W;
  static_assert(4 * W * sizeof(C2<R>) == 128, "128-byte stencil blocks");
  typedef R R2 __attribute__((ext_vector_type(2)));
  typedef float F4 __attribute__((ext_vector_type(4)));
  R w[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g) lagrange4(sfr[K0 + g], w[g]);
  C2<R> Z[G];
#pragma unroll
  for (int g = 0; g < G; ++g) Z[g].x = Z[g].y = 0;
  C2<R> ph;
  ph.x = 1;
  ph.y = 0;
  const int mmin = P->m_min;
  for (int t = 0; t < -mmin; ++t) phase_down(ph, cf, sf);
  int mc = mmin < 0 ? mmin : 0;
  // Y of the W modes of group p; the slots past M repeat mode M-1 (their
  // taps are zero, so they add exact zeros)
  R yx[W], yy[W];
  auto ycomp = [&](int p) {
#pragma unroll
    for (int s = 0; s < W; ++s) {
      const int i = p * W + s;
      const int ic = i < M ? i : M - 1;
      const int mi = P->m[ic];
      while (mc < mi) {
        phase_up(ph, cf, sf);
        ++mc;
      }
      const R d = mode_d<R, NY>(P, ic, cn, sn);
      yx[s] = d * ph.x;
      yy[s] = d * ph.y;
    }
  };
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int q = lane >> 3;
  // key(8 t + q) = ((t & 1) << 2) | (q >> 1): the chunk offsets of even and odd reads
  const uint32_t cx0 = (uint32_t)((lane & 7) ^ (q >> 1)) << 4;
  const uint32_t cx1 = (uint32_t)((lane & 7) ^ (4 | (q >> 1))) << 4;
  // read t of detector g: this lane's source offset
  uint32_t offt[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int t = 0; t < 8; ++t) offt[g][t] = (uint32_t)__shfl((int)boff[K0 + g], 8 * t + q) + ((t & 1) ? cx1 : cx0);
  // chunk c of this lane's block: rbase ^ (c << 4)
  const uint32_t rbase = (uint32_t)lane * 128u + ((uint32_t)((lane >> 1) & 7) << 4);
  auto issue = [&](int p, int g, int b) {
    const RIFT_GLOBAL char* ser = uniform_ptr(Qb + (uint64_t)(K0 + g) * kstride + (uint64_t)p * gstride);
    RIFT_LDS unsigned char* dst = stage + b * STAGE_UNIT;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      __builtin_amdgcn_global_load_lds((const RIFT_GLOBAL void*)(ser + offt[g][t]), (RIFT_LDS void*)(dst + t * 1024),
                                       16, 0, 0);
  };
  auto consume = [&](int b, int g) {
    const RIFT_LDS unsigned char* src = stage + b * STAGE_UNIT;
    C2<R> u[4][W];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t a = rbase ^ ((uint32_t)c << 4);
      if constexpr (sizeof(R) == 8) {
        const R2 v = *(const RIFT_LDS R2*)(src + a);
        u[c >> 1][c & 1].x = v.x;
        u[c >> 1][c & 1].y = v.y;
      } else {
        const F4 v = *(const RIFT_LDS F4*)(src + a);
        u[c >> 1][2 * (c & 1)].x = v.x;
        u[c >> 1][2 * (c & 1)].y = v.y;
        u[c >> 1][2 * (c & 1) + 1].x = v.z;
        u[c >> 1][2 * (c & 1) + 1].y = v.w;
      }
    }
#pragma unroll
    for (int s = 0; s < W; ++s) mode_acc(Z[g], w[g], u[0][s], u[1][s], u[2][s], u[3][s], yx[s], yy[s]);
    // the unit is combined here, before the next refill is issued (instead
    // of its FMAs sinking past later units, keeping their reads live)
    pin(Z[g].x);
    pin(Z[g].y);
  };
  // Unit u = p G + g uses buffer u & 1; an iteration covers an even number of
  // units, so every buffer index is a constant.  Each buffer is refilled only
  // after the LDS reads of its previous unit have completed, and a unit is
  // read only after its own global reads have (the newer unit's eight reads
  // may still be in flight).
  constexpr int UPI = (G % 2 == 0) ? G : 2 * G;
  const int total = NGR * G;
  issue(0, 0, 0);
#pragma unroll 1
  for (int p0 = 0; p0 < NGR; p0 += UPI / G) {
#pragma unroll
    for (int v = 0; v < UPI; ++v) {
      const int p = p0 + v / G;
      const int g = v % G;
      if (g == 0 && p >= NGR) break;
      if (p * G + g + 1 < total) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(g + 1 == G ? p + 1 : p, (g + 1) % G, (v + 1) & 1);
        if (g == 0) ycomp(p);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      } else {
        if (g == 0) ycomp(p);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      consume(v & 1, g);
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  double acc = 0.0;
#pragma unroll
  for (int g = 0; g < G; ++g)
    acc += (double)(Fre[K0 + g] * Z[g].x) + (double)(Fim[K0 + g] * Z[g].y);
  if constexpr (CPLX) {
    double ai = 0.0;
#pragma unroll
    for (int g = 0; g < G; ++g) ai += (double)(Fre[K0 + g] * Z[g].y) - (double)(Fim[K0 + g] * Z[g].x);
    *acc_im += ai;
  }
  return acc;
}

// Data term of one sample from a table of short rows.
template <class R, int KT, int L, bool CPLX = false>
__device__ __forceinline__ double data_direct(PDesc P, RIFT_LDS unsigned char* stage, const int32_t* row,
                                              const R* sfr, const R* Fre, const R* Fim, const R* cn,
                                              const R* sn, R cf, R sf, double* im = nullptr) {
  static_assert(KT >= 2, "detector counts are padded to at least two");
  constexpr int NY = Cls<L>::NY;
  constexpr int W = Tab<R>::W;
  const int M = P->M;
  const int NGR = q_groups(M, W);
  uint32_t boff[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) boff[k] = (uint32_t)row[k] * (uint32_t)(W * sizeof(C2<R>));
  const RIFT_GLOBAL char* Qb = (const RIFT_GLOBAL char*)Tab<R>::Q(P);
  const uint64_t gstride = (uint64_t)(P->n_t + 2 * QPAD) * (W * sizeof(C2<R>));
  const uint64_t kstride = (uint64_t)NGR * gstride;
  constexpr int G0 = det_group_size(KT, 0), G1 = det_group_size(KT, 1), G2 = det_group_size(KT, 2);
  double data = data_group<R, NY, 0, G0, CPLX>(P, Qb, gstride, kstride, M, NGR, boff, stage, sfr, Fre, Fim, cn,
                                               sn, cf, sf, im);
  if constexpr (G1 > 0)
    data += data_group<R, NY, det_group_start(KT, 1), G1, CPLX>(P, Qb, gstride, kstride, M, NGR, boff, stage, sfr,
                                                                Fre, Fim, cn, sn, cf, sf, im);
  if constexpr (G2 > 0)
    data += data_group<R, NY, det_group_start(KT, 2), G2, CPLX>(P, Qb, gstride, kstride, M, NGR, boff, stage, sfr,
                                                                Fre, Fim, cn, sn, cf, sf, im);
  return data;
}

// The model-norm contraction of FP64 (up to three detectors) in steps, for
// interleaving with the data term's reads: acc[c] = sum_b C[b][c] beta_b(incl, phi),
// the rows of the basis in pairs of one degree n and phase q,
//   q = 0: (T_n, T_n+1), n = 1, 3, ..;  q >= 1: T_n (cos q phi, sin q phi),
// T_n = cos(n incl) for even q and sin(n incl) for odd q, from three-term
// recurrences in n: no table of the harmonics is kept.  A cycle is the pairs of
// an odd and the next even q, unrolled; step<S> takes RPS rows of the cycle,
// whose coefficients were loaded into SGPRs one step ahead.
template <int KT, int L>
struct NormWalk {
  static constexpr int NI = 2 * L, W = 3 * KT;
  static constexpr int PAIRS = 2 * NI + 1, CYCLES = NI / 2;
  static constexpr int RPS = KT == 2 ? 4 : 2;                // at most 48 SGPRs (KT <= 3)
  static constexpr int STEPS = (2 * PAIRS + RPS - 1) / RPS;  // the last may be short
  static_assert(Cls<L>::B == 1 + NI + 2 * CYCLES * PAIRS, "row 0, the pairs of q = 0, and the cycles");
  static constexpr int rows(int S, int all) { return all - S * RPS < RPS ? all - S * RPS : RPS; }
  const RIFT_CONST double* C;
  double buf[RPS * W];
  double bx, by, px, py;  // the pair's values, and those before
  double ex, ey;          // e^{i q phi}
  double ci, si, cf, sf;

  template <int ROWS>
  __device__ __forceinline__ void load() {
    const RIFT_CONST double* p = opaque(C);
#pragma unroll
    for (int i = 0; i < ROWS * W; ++i) buf[i] = p[i];
  }
  template <int ROWS>
  __device__ __forceinline__ void wait() {
#pragma unroll
    for (int i = 0; i < ROWS * W; ++i) pin_s(buf[i]);
  }
  __device__ __forceinline__ void add(int row, double b, double* acc) {
#pragma unroll
    for (int c = 0; c < W; ++c) acc[c] = fma(buf[row * W + c], b, acc[c]);
  }
  template <int ROWS, int NEXT>
  __device__ __forceinline__ void done(double* acc) {
#pragma unroll
    for (int c = 0; c < W; ++c) pin(acc[c]);
    C += ROWS * W;
    load<NEXT>();
  }
  // step S of the rows after row 0 with q = 0
  template <int S>
  __device__ __forceinline__ void first(double* acc) {
    if constexpr (S * RPS < NI) {
      constexpr int N = rows(S, NI);
      wait<N>();
#pragma unroll
      for (int r = 0; r < N; ++r) {
        add(r, bx, acc);
        const double t = fma(2.0 * ci, bx, -px);
        px = bx;
        bx = t;
      }
      done<N, (S + 1) * RPS < NI ? rows(S + 1, NI) : rows(0, 2 * PAIRS)>(acc);
      first<S + 1>(acc);
    }
  }
  __device__ __forceinline__ void start(const RIFT_CONST double* C0, double ci_, double si_, double cf_, double sf_,
                                        double* acc) {
    ci = ci_;
    si = si_;
    cf = cf_;
    sf = sf_;
    C = C0 + W;
    load<rows(0, NI)>();
#pragma unroll
    for (int c = 0; c < W; ++c) acc[c] = C0[c];
    bx = ci;
    px = 1.0;
    first<0>(acc);
    ex = 1.0;
    ey = 0.0;
  }
  __device__ __forceinline__ void turn() {
    const double t = ex * cf - ey * sf;
    ey = ex * sf + ey * cf;
    ex = t;
  }
  // pair J of the cycle's
  template <int J>
  __device__ __forceinline__ void pair() {
    if constexpr (J == 0) {
      turn();
      bx = si * ex;
      by = si * ey;
      px = py = 0.0;
    } else if constexpr (J == NI) {
      turn();
      bx = ex;
      by = ey;
      px = ci * ex;
      py = ci * ey;
    } else {
      const double x = fma(2.0 * ci, bx, -px), y = fma(2.0 * ci, by, -py);
      px = bx;
      py = by;
      bx = x;
      by = y;
    }
  }
  template <int S>
  __device__ __forceinline__ void step(double* acc, bool last) {
    constexpr int N = rows(S, 2 * PAIRS);
    wait<N>();
    pair<S * RPS / 2>();
    add(0, bx, acc);
    add(1, by, acc);
    if constexpr (N == 4) {
      pair<S * RPS / 2 + 1>();
      add(2, bx, acc);
      add(3, by, acc);
    }
    if constexpr (S + 1 < STEPS) {
      done<N, rows(S + 1, 2 * PAIRS)>(acc);
    } else {  // the next cycle's; the last reads its own rows again
      static_assert(rows(0, 2 * PAIRS) >= N, "a short step is read again in part of a whole one");
      if (last) C -= (rows(0, 2 * PAIRS) - N) * W + N * W;
      done<N, rows(0, 2 * PAIRS)>(acc);
    }
  }
  // steps A .. B - 1
  template <int A, int B>
  __device__ __forceinline__ void steps(double* acc, bool last) {
    if constexpr (A < B) {
      step<A>(acc, last);
      steps<A + 1, B>(acc, last);
    }
  }
};
// The detector counts that walk: the accumulators and antenna factors of five spill
// beside the reads (5 detectors, 21 modes, 3e5 samples: 198 us with the walk, 189
// with the contraction after the reads).
constexpr bool walks(int KT) { return KT <= 3; }
constexpr int WALK_GROUPS = 2;  // groups of eight modes (of one detector) per cycle

// The modes of a group of eight, two per unit of the group's first detector:
// their coefficients are loaded (fetch) before the unit's share of the norm and
// used (take(slot, m, d_i(incl))) after it.
template <int NY>
struct ModeWalk {
  double c[2][NY];
  int m[2], odd[2];
  __device__ __forceinline__ void fetch(PDesc P, int i0, int M) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = i0 + j < M ? i0 + j : M - 1;  // the slots past M repeat it (their taps are zero)
      m[j] = P->m[i];
      odd[j] = P->odd[i];
#pragma unroll
      for (int n = 0; n < NY; ++n) c[j][n] = P->ycoef[i][n];
    }
  }
  // d_i(incl) from cos incl and sin incl alone (Clenshaw's recurrence): no
  // table of the harmonics is kept through the reads
  __device__ __forceinline__ double d(int j, double ci, double si) const {
    const double c2 = 2.0 * ci;
    double b1 = 0.0, b2 = 0.0;
#pragma unroll
    for (int n = NY - 1; n >= 1; --n) {
      const double b = fma(c2, b1, c[j][n] - b2);
      b2 = b1;
      b1 = b;
    }
    return odd[j] ? si * b1 : fma(ci, b1, c[j][0] - b2);
  }
};

// The FP64 reads of the data term, detector by detector in each group of eight
// modes.
//
// The unit is one aligned 128-byte line per lane, one stencil row of a group:
// every line that a read brings into the vector cache is used whole (blocks of
// four rows of two modes straddled two lines three times in four: 19.25 lines a
// sample and detector at 21 modes, where this reads 12).  The lines are read
// cooperatively, straight to LDS: eight lanes fetch the eight 16-byte chunks of
// one lane's line, so that a read instruction touches 8 lines.  Lane
// l = 8 q + c' of read t fetches chunk c = c' ^ key(j) of the line of lane
// j = 8 t + q, which lands at j * 128 + c' * 16; with key(j) = (j >> 1) & 7
// the eight lanes of equal j * 128 mod 256 within any sixteen consecutive lanes
// read eight different 16-byte columns, so lane j's own reads of its chunks
// are free of bank conflicts.
//
// Units stream through the wavefront's two LDS buffers: unit u + 1 is in
// flight while unit u is combined.  The whole wavefront calls this together.
// Offsets are 32-bit, so a table is read in windows of 2^24 rows: one, but for
// the longest.
constexpr int ROWS_WINDOW = 1 << 24;
typedef double Cplx __attribute__((ext_vector_type(2)));
template <int KT, int W>
struct RowReader {
  static constexpr int UNITS = W / 2;                        // of a group: of 4 / UNITS rows each
  static constexpr uint32_t ROW = W * sizeof(C2<double>);    // bytes
  static constexpr int LAST = UNITS - 1;
  static_assert(4 * ROW == 128 * UNITS && (W == QW64 || W == QW64_SHORT), "units of 128 bytes");
  static constexpr uint32_t BIAS = 3072;
  PDesc P;
  const int32_t* row;
  RIFT_LDS unsigned char* lds;
  const RIFT_GLOBAL char *series, *first, *next;  // this group, detector 0's, and the next
  uint64_t kstride, gstride;
  uint32_t off[8], rbase;
  int K, window, left, k, p;  // left: groups of all detectors still to come, this one included
  int flip;                   // the buffer of a group's first unit (0 where a group has four)

  __device__ __forceinline__ void offsets(int kk) {
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int q = lane >> 3;
    // key(8 t + q) = ((t & 1) << 2) | (q >> 1): the chunks of even and odd reads
    const uint32_t cx0 = (uint32_t)((lane & 7) ^ (q >> 1)) << 4;
    const uint32_t r = (uint32_t)(by_det<KT>(row, kk) - window);
    const uint32_t b = (r < (uint32_t)ROWS_WINDOW ? r : 0u) * ROW + BIAS;
    // read t's immediate offset, (t & 3) KB, goes to both addresses: the
    // source offsets are biased by the largest
#pragma unroll
    for (int t = 0; t < 8; ++t)
      off[t] = (uint32_t)__shfl((int)b, 8 * t + q) + ((t & 1) ? cx0 ^ 64u : cx0) - (uint32_t)(t & 3) * 1024u;
  }
  __device__ __forceinline__ void issue(const RIFT_GLOBAL char* from, int tap) {
    const RIFT_GLOBAL char* ser = uniform_ptr(from + (tap % UNITS) * 128 - BIAS);
    RIFT_LDS unsigned char* dst = lds + ((tap + flip) & 1) * STAGE_UNIT;
#define RIFT_READ(t) \
  __builtin_amdgcn_global_load_lds((const RIFT_GLOBAL void*)(ser + off[t]), (RIFT_LDS void*)(dst + (t & 4) * 1024), 16, \
                                   (t & 3) * 1024, 0)
    RIFT_READ(0);
    RIFT_READ(1);
    RIFT_READ(2);
    RIFT_READ(3);
    RIFT_READ(4);
    RIFT_READ(5);
    RIFT_READ(6);
    RIFT_READ(7);
#undef RIFT_READ
  }
  __device__ __forceinline__ void start(PDesc P_, RIFT_LDS unsigned char* stage, const int32_t* row_, int window_) {
    P = P_;
    row = row_;
    window = window_;
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    // chunk c of this lane's line: rbase ^ (c << 4)
    lds = (RIFT_LDS unsigned char*)(uintptr_t)(uint32_t)uniform_i((int)(uintptr_t)stage);
    rbase = (uint32_t)lane * 128u + ((uint32_t)((lane >> 1) & 7) << 4);
    K = P->K;
    const int NGR = q_groups(P->M, W);
    left = K * NGR;
    flip = 0;
    gstride = (uint64_t)(P->n_t + 2 * QPAD) * ROW;
    kstride = (uint64_t)NGR * gstride;
    series = first = (const RIFT_GLOBAL char*)as_global(P->Q64) + (uint64_t)(uint32_t)window * ROW;
    k = p = 0;
    offsets(0);
    issue(series, 0);
  }
  // Before unit `tap` of the current group is combined: the next unit's reads.
  __device__ __forceinline__ void ahead(int tap) {
    // the other buffer's values are in registers already
    asm volatile("" ::: "memory");
    if (tap == 0) next = k + 1 < K ? series + kstride : first + gstride;
    if (tap < LAST) {
      issue(series, tap + 1);
    } else if (left > 1) {
      if constexpr (UNITS == 1) offsets(k + 1 < K ? k + 1 : 0);
      issue(next, UNITS);
    }
  }
  // Unit `tap` of the current group.
  __device__ __forceinline__ void fetch(int tap, Cplx* v) {
    // the newer unit's eight reads may still be in flight
    if (tap == LAST && left == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    if (UNITS > 1 && tap == LAST - 1 && left > 1) offsets(k + 1 < K ? k + 1 : 0);
    const RIFT_LDS unsigned char* src = lds + ((tap + flip) & 1) * STAGE_UNIT;
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = *(const RIFT_LDS Cplx*)(src + (rbase ^ ((uint32_t)c << 4)));
    // all of them at once, in registers before the buffer's next refill
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])
                 :
                 : "memory");
  }
  __device__ __forceinline__ void advance() {
    --left;
    if (UNITS & 1) flip ^= 1;
    series = next;
    if (++k == K) {
      k = 0;
      ++p;
      first = next;
    }
  }
};
// Whether a sample's stencil starts in the window of rows.
__device__ __forceinline__ bool in_window(int32_t row, int window) {
  return (uint32_t)(row - window) < (uint32_t)ROWS_WINDOW;
}

// The data term of one sample in FP64 and, with NORM, the model-norm contraction
// acc (see NormWalk) in the shadow of its reads.  Y_i = d_i(incl) e^{i m_i phi};
// the modes are sorted by m, so the phase walks upward from e^{i m_min phi}.
// With CPLX, the imaginary part goes to *im.
template <int KT, int L, bool NORM, bool CPLX>
struct DataNorm {
  static constexpr int W = QW64;
  static constexpr int UNITS = RowReader<KT, W>::UNITS;
  PDesc P;
  const int32_t* row;
  const double *sfr, *Fre, *Fim;
  double* acc;
  double ci, si, cf, sf;
  double re, im;
  RowReader<KT, W> R;
  NormWalk<KT, L> walk;
  ModeWalk<L + 1> mode;
  C2<double> ph;
  int mc;
  double w[4], yx[W], yy[W], qx[W], qy[W];

  __device__ __forceinline__ void modes(int t) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      while (mc < mode.m[j]) {
        phase_up(ph, cf, sf);
        ++mc;
      }
      const double d = mode.d(j, ci, si);
      yx[2 * t + j] = d * ph.x;
      yy[2 * t + j] = d * ph.y;
    }
  }
  __device__ __forceinline__ void take(int t) {
    Cplx v[8];
    R.fetch(t, v);
#pragma unroll
    for (int c = 0; c < 8; ++c) {  // row t 8 / W + c / W of the stencil, mode c % W
      const int r = t * (8 / W) + c / W, s = c % W;
      qx[s] = r == 0 ? w[r] * v[c].x : fma(w[r], v[c].x, qx[s]);
      qy[s] = r == 0 ? w[r] * v[c].y : fma(w[r], v[c].y, qy[s]);
      pin(qx[s]);
      pin(qy[s]);
    }
  }
  __device__ __forceinline__ void fold() {
    double zr = 0.0, zi = 0.0;
#pragma unroll
    for (int s = 0; s < W; ++s) {
      zr = fma(yx[s], qx[s], zr);
      zr = fma(yy[s], qy[s], zr);
      zi = fma(yx[s], qy[s], zi);
      zi = fma(-yy[s], qx[s], zi);
    }
    if (P->n_t + 2 * QPAD > ROWS_WINDOW && !in_window(by_det<KT>(row, R.k), R.window)) zr = zi = 0.0;
    const double fr = by_det<KT>(Fre, R.k), fi = by_det<KT>(Fim, R.k);
    re = fma(fr, zr, re);
    re = fma(fi, zi, re);
    if constexpr (CPLX) {
      im = fma(fr, zi, im);
      im = fma(-fi, zr, im);
      pin(im);
    }
    pin(re);
    R.advance();
  }
  // Unit u of a cycle's, with the cycle's steps spread over both halves of the
  // units (CYCLE), or alone.
  template <int U, int N, bool CYCLE>
  __device__ __forceinline__ void unit(bool last) {
    constexpr int T = U % UNITS, S = NormWalk<KT, L>::STEPS;
    if (!CYCLE || R.left > 0) {
      if constexpr (T == 0) lagrange4(by_det<KT>(sfr, R.k), w);
      R.ahead(T);
      if (R.k == 0) mode.fetch(P, R.p * W + 2 * T, P->M);
    }
    if constexpr (CYCLE) walk.template steps<2 * U * S / (2 * N), (2 * U + 1) * S / (2 * N)>(acc, last);
    if (!CYCLE || R.left > 0) {
      if (R.k == 0) modes(T);
      take(T);
    }
    if constexpr (CYCLE) walk.template steps<(2 * U + 1) * S / (2 * N), (2 * U + 2) * S / (2 * N)>(acc, last);
    if (T == UNITS - 1 && (!CYCLE || R.left > 0)) fold();
  }
  template <int U, int N, bool CYCLE>
  __device__ __forceinline__ void units(bool last) {
    if constexpr (U < N) {
      unit<U, N, CYCLE>(last);
      units<U + 1, N, CYCLE>(last);
    }
  }
  __device__ __forceinline__ void run(RIFT_LDS unsigned char* stage) {
    const int rows = P->n_t + 2 * QPAD;
    re = im = 0.0;
#pragma unroll 1
    for (int window = 0; window < rows; window += ROWS_WINDOW) {
      R.start(P, stage, row, window);
      ph.x = 1.0;
      ph.y = 0.0;
      const int mmin = P->m_min;
      for (int t = 0; t < -mmin; ++t) phase_down(ph, cf, sf);
      mc = mmin < 0 ? mmin : 0;
      if constexpr (NORM) {
        if (window == 0) {
          walk.start(as_const(P->C64), ci, si, cf, sf, acc);
#pragma unroll 1
          for (int it = 0; it < NormWalk<KT, L>::CYCLES; ++it)
            units<0, UNITS * WALK_GROUPS, true>(it + 1 == NormWalk<KT, L>::CYCLES);
        }
      }
#pragma unroll 1
      while (R.left > 0) units<0, UNITS, false>(false);
    }
  }
};
template <int KT, int L, bool NORM, bool CPLX>
__device__ __forceinline__ double data_rows(PDesc P, RIFT_LDS unsigned char* stage, const int32_t* row,
                                            const double* sfr, const double* Fre, const double* Fim,
                                            double ci, double si, double cf, double sf, double* acc, double* im) {
  DataNorm<KT, L, NORM, CPLX> D;
  D.P = P;
  D.row = row;
  D.sfr = sfr;
  D.Fre = Fre;
  D.Fim = Fim;
  D.acc = acc;
  D.ci = ci;
  D.si = si;
  D.cf = cf;
  D.sf = sf;
  D.run(stage);
  if constexpr (CPLX) *im = D.im;
  return D.re;
}
// Result of one sample evaluation.
struct Eval {
  double lnL;
  float bound;  // a-priori |lnL - lnL_FP64| bound (FP32 arithmetic only)
};

// Antenna factors of one sample and, for the data term, its stencils: the sky
// frame (FP64), the polarisation tensors and F_k = F+ + i Fx (R), and per
// detector the arrival time t_k and stencil row / fraction (FP64 phase).
template <class R, int KT>
struct Sky {
  R Fre[KT], Fim[KT];
  R sfr[KT];        // fractional position inside the stencil cell
  int32_t row[KT];  // padded index of the first stencil row, in [0, n_t + QPAD]
  bool bad;         // a non-finite arrival time
  double N[3];      // direction to the source
};
// The stencils of every detector for geocentric time t (the sky frame in S).
template <class R, int KT>
__device__ __forceinline__ void sky_stencils(PDesc P, double t, Sky<R, KT>& S) {
  const int n_t = P->n_t;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const RIFT_CONST double* r = P->rpos[k];
    const double tk = t - (r[0] * S.N[0] + r[1] * S.N[1] + r[2] * S.N[2]);
    double u = (tk - P->t0) * P->inv_dt;
    if (!stencil_u(u, n_t)) S.bad = true;
    const double jf = floor(u);
    const R s = (R)(u - jf);
    int j0 = (int)jf - 1;  // stencil rows j0 .. j0+3
    // wholly outside the stored window: read four zero pad rows
    j0 = j0 < -QPAD ? -QPAD : (j0 > n_t ? n_t : j0);
    S.row[k] = j0 + QPAD;
    S.sfr[k] = s;
  }
}
// (sin, cos) of incl and phi, which the harmonics take, come out with them.
template <class R, int KT, bool STENCIL>
__device__ __forceinline__ void sky_eval(PDesc P, double ra, double dec, double psi, double incl, double phi,
                                         double tref, Sky<R, KT>& S, R& si, R& ci, R& sf, R& cf) {
  double sg, cg, sd, cd;
  R sp, cp;
  if constexpr (sizeof(R) == 8) {
    const double a[5] = {P->gmst - ra, dec, psi, incl, phi};
    double s[5], c[5];
    sincos_many<5>(a, s, c);
    sg = s[0];
    cg = c[0];
    sd = s[1];
    cd = c[1];
    sp = s[2];
    cp = c[2];
    si = s[3];
    ci = c[3];
    sf = s[4];
    cf = c[4];
  } else {
    const double a[2] = {P->gmst - ra, dec};
    double s[2], c[2];
    sincos_many<2>(a, s, c);
    sg = s[0];
    cg = c[0];
    sd = s[1];
    cd = c[1];
    sincosf((R)psi, &sp, &cp);
    sincosf((R)incl, &si, &ci);
    sincosf((R)phi, &sf, &cf);
  }
  const double N0 = cd * cg, N1 = -cd * sg, N2 = sd;
  S.N[0] = N0;
  S.N[1] = N1;
  S.N[2] = N2;
  const R ea0 = (R)sg, ea1 = (R)cg;
  const R ed0 = (R)(-sd * cg), ed1 = (R)(sd * sg), ed2 = (R)cd;
  const R X0 = -cp * ea0 + sp * ed0, X1 = -cp * ea1 + sp * ed1, X2 = sp * ed2;
  const R Y0 = sp * ea0 + cp * ed0, Y1 = sp * ea1 + cp * ed1, Y2 = cp * ed2;
  const R ep[6] = {X0 * X0 - Y0 * Y0, X1 * X1 - Y1 * Y1, X2 * X2 - Y2 * Y2,
                   X0 * X1 - Y0 * Y1, X0 * X2 - Y0 * Y2, X1 * X2 - Y1 * Y2};
  const R ex[6] = {2 * X0 * Y0, 2 * X1 * Y1, 2 * X2 * Y2,
                   X0 * Y1 + Y0 * X1, X0 * Y2 + Y0 * X2, X1 * Y2 + Y1 * X2};
  S.bad = false;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    R fp = 0, fx = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
      fp += Tab<R>::d(P, k, a) * ep[a];
      fx += Tab<R>::d(P, k, a) * ex[a];
    }
    S.Fre[k] = fp;
    S.Fim[k] = fx;
  }
  if constexpr (STENCIL) sky_stencils<R, KT>(P, tref, S);
}

// The angles that the FP32 arithmetic takes, reduced in FP64 first.
template <class R>
__device__ __forceinline__ void reduce_angles(double& psi, double& incl, double& phi) {
  if constexpr (sizeof(R) == 4) {
    psi = reduce_2pi(psi);
    incl = reduce_2pi(incl);
    phi = reduce_2pi(phi);
  }
}

// Model-norm term sum_k |F_k|^2 a_k/4 + Re(F_k^2 b_k)/4 from the basis
// contraction at (incl, phiref); with BOUND, also the model-norm part of the
// FP32 error bound (see PointDesc).  `trig` is this lane's column of a
// block-shared scratch array (stride `ts` elements) that receives
// cos(n incl), n = 0..NI, then sin(n incl), for the runtime contraction loop
// of the l <= 8 class.
template <class R, int KT, int L>
__device__ __forceinline__ void norm_contract(PDesc P, R* __restrict__ trig, int ts, R ci, R si, R cf, R sf,
                                              R* acc) {
  typedef Cls<L> CL;
  constexpr int NI = CL::NI;
#pragma unroll
  for (int c = 0; c < 3 * KT; ++c) acc[c] = 0;
  if constexpr (L <= 4) {
    Contract<R, KT, L>::run(P, ci, si, cf, sf, acc);
  } else {
    {
      R c0 = 1, c1 = ci, s0 = 0, s1 = si;
#pragma unroll
      for (int n = 0; n <= NI; ++n) {
        trig[n * ts] = (n == 0) ? c0 : c1;
        trig[(NI + 1 + n) * ts] = (n == 0) ? s0 : s1;
        if (n > 0) {
          const R c2 = 2 * ci * c1 - c0, s2 = 2 * ci * s1 - s0;
          c0 = c1;
          c1 = c2;
          s0 = s1;
          s1 = s2;
        }
      }
    }
    // runtime loop over basis rows (reads cos/sin(n incl) from this lane's
    // column of the block-shared scratch array)
    const RIFT_CONST R* Cc = Tab<R>::C(P);
    {
      // q = 0: rows n = 0..NI, basis cos(n incl)
      R cur[3 * KT];
#pragma unroll
      for (int c = 0; c < 3 * KT; ++c) cur[c] = Cc[c];
      R tcur = trig[0];
#pragma unroll 1
      for (int n = 0; n <= NI; ++n) {
        const int nn = (n < NI) ? n + 1 : n;
        R nxt[3 * KT];
#pragma unroll
        for (int c = 0; c < 3 * KT; ++c) nxt[c] = Cc[nn * 3 * KT + c];
        const R tnxt = trig[nn * ts];
#pragma unroll
        for (int c = 0; c < 3 * KT; ++c) acc[c] = fma(cur[c], tcur, acc[c]);
#pragma unroll
        for (int c = 0; c < 3 * KT; ++c) cur[c] = nxt[c];
        tcur = tnxt;
      }
    }
    {
      // q >= 1: pairs of rows (T_n cos(q phi), T_n sin(q phi)); even q pairs
      // with cos(n incl) for n = 0..NI, odd q with sin(n incl) for n = 1..NI
      const int B = CL::B;
      int b = NI + 1;
      C2<R> eq;
      eq.x = cf;
      eq.y = sf;
      R cur[6 * KT];
#pragma unroll
      for (int c = 0; c < 6 * KT; ++c) cur[c] = Cc[b * 3 * KT + c];
#pragma unroll 1
      for (int q = 1; q <= NI; ++q) {
        const int odd = q & 1;
        const int base = odd ? (NI + 1) : 0;
        R tcur = trig[(base + odd) * ts];
#pragma unroll 1
        for (int n = odd; n <= NI; ++n, b += 2) {
          // next pair of rows (the last iteration re-reads its own rows)
          const int bn = (b + 2 < B) ? b + 2 : b;
          R nxt[6 * KT];
#pragma unroll
          for (int c = 0; c < 6 * KT; ++c) nxt[c] = Cc[bn * 3 * KT + c];
          const int tn = (n < NI) ? base + n + 1 : base + n;
          const R tnxt = trig[tn * ts];
          const R b1 = tcur * eq.x, b2 = tcur * eq.y;
#pragma unroll
          for (int c = 0; c < 3 * KT; ++c) {
            acc[c] = fma(cur[c], b1, acc[c]);
            acc[c] = fma(cur[3 * KT + c], b2, acc[c]);
          }
#pragma unroll
          for (int c = 0; c < 6 * KT; ++c) cur[c] = nxt[c];
          tcur = tnxt;
        }
        const R ex_ = eq.x * cf - eq.y * sf, ey_ = eq.x * sf + eq.y * cf;
        eq.x = ex_;
        eq.y = ey_;
      }
    }
  }
}

template <class R, int KT, bool BOUND>
__device__ __forceinline__ double quad_of(PDesc P, const R* acc, const R* Fre, const R* Fim, double* wq_out) {
  double quad = 0.0;
  double wq = 0.0;  // model-norm part of the error bound (see PointDesc)
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const R f2 = Fre[k] * Fre[k] + Fim[k] * Fim[k];
    const R g2r = Fre[k] * Fre[k] - Fim[k] * Fim[k];
    const R g2i = 2 * Fre[k] * Fim[k];
    quad += (double)(f2 * acc[3 * k]) + (double)(g2r * acc[3 * k + 1]) +
            (double)(g2i * acc[3 * k + 2]);
    if (BOUND) {
      const double e = P->eF[k];
      const double fe = sqrt((double)f2) + e;  // >= |F_k| of the exact arithmetic
      wq += fe * fe * P->bnd_q[k] + (2.0 * fe + e) * e * P->l1q[k];
    }
  }
  if (BOUND) *wq_out = wq;
  return quad;
}
template <class R, int KT, int L, bool BOUND>
__device__ __forceinline__ double quad_term(PDesc P, R* __restrict__ trig, int ts, R ci, R si, R cf, R sf,
                                            const R* Fre, const R* Fim, double* wq_out) {
  R acc[3 * KT];
  norm_contract<R, KT, L>(P, trig, ts, ci, si, cf, sf, acc);
  return quad_of<R, KT, BOUND>(P, acc, Fre, Fim, wq_out);
}

// cos(n incl), sin(n incl) for n < NY by the Chebyshev recurrences.
template <class R, int NY>
__device__ __forceinline__ void incl_harmonics(R ci, R si, R* cn, R* sn) {
  R c0 = 1, c1 = ci, s0 = 0, s1 = si;
#pragma unroll
  for (int n = 0; n < NY; ++n) {
    cn[n] = (n == 0) ? c0 : c1;
    sn[n] = (n == 0) ? s0 : s1;
    if (n > 0) {
      const R c2 = 2 * ci * c1 - c0, s2 = 2 * ci * s1 - s0;
      c0 = c1;
      c1 = c2;
      s0 = s1;
      s1 = s2;
    }
  }
}

// The data term of one sample in FP64 and, with NORM, the model-norm contraction
// acc: by rows where they hold eight modes, up to three detectors with the
// contraction between the units; otherwise one after the other.
template <int KT, int L, bool NORM, bool CPLX>
__device__ __forceinline__ double data_norm(PDesc P, double* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                            const int32_t* row, const double* sfr, const double* Fre,
                                            const double* Fim, double ci, double si, double cf, double sf, double* acc,
                                            double* im) {
  double data;
  if constexpr (Cls<L>::MAXM > QW64_SHORT_MODES) {
    if (P->w64 == QW64) {
      __builtin_amdgcn_s_setprio(1);
      data = data_rows<KT, L, NORM && walks(KT), CPLX>(P, stage, row, sfr, Fre, Fim, ci, si, cf, sf, acc, im);
      __builtin_amdgcn_s_setprio(0);
      if constexpr (NORM && !walks(KT)) norm_contract<double, KT, L>(P, trig, ts, ci, si, cf, sf, acc);
      return data;
    }
  }
  constexpr int NY = Cls<L>::NY;
  double cn[NY], sn[NY];
  incl_harmonics<double, NY>(ci, si, cn, sn);
  if constexpr (CPLX) *im = 0.0;
  __builtin_amdgcn_s_setprio(1);
  data = data_direct<double, KT, L, CPLX>(P, stage, row, sfr, Fre, Fim, cn, sn, cf, sf, im);
  __builtin_amdgcn_s_setprio(0);
  if constexpr (NORM) norm_contract<double, KT, L>(P, trig, ts, ci, si, cf, sf, acc);
  return data;
}

// lnL = x data - x^2 quad with x = D_ref / D (FP64), NaN for a poisoned
// sample, and the a-priori FP32 bound |x| bnd_d + x^2 wq, rounded up on the
// way to FP32 (the factor covers the conversion).
template <bool BOUND>
__device__ __forceinline__ Eval combine(PDesc P, double dist, double data, double quad, double wq, bool bad) {
  const double x = P->d_ref / dist;
  Eval e;
  e.lnL = x * data - x * x * quad;
  if (bad) e.lnL = __builtin_nan("");
  e.bound = 0.0f;
  if (BOUND) e.bound = (float)((fabs(x) * P->bnd_d + x * x * wq) * (1.0 + 1.0e-6));
  return e;
}

// The distance-free terms of one sample: lnL(x) = x data - x^2 quad with
// x = D_ref / D; wq is the model-norm part of the FP32 bound (BOUND only).
struct Terms {
  double data, quad, wq;
  bool bad;
};

// Gauss-Hermite rule of the distance marginal (weight e^{-xi^2/2}; up to
// DM_MAX nodes) and the prior p(D) proportional to D^2 on [d_min, d_max].
constexpr int DM_MAX = 64;
struct DistRule {
  int32_t n;
  int32_t pad;
  double d_min, d_max;
  double ln_norm;  // ln(3 / (d_max^3 - d_min^3))
  double xi[DM_MAX], w[DM_MAX];
};

// ln of the likelihood marginalised over distance, Eq. (ap:dgh), from the
// terms: with lnL(x) = K x - R x^2 / 2 (K = data, R = 2 quad), the peak
// x* = K / R and width sigma = R^-1/2 of Eq. (ap:dpeak) centre and scale the
// nodes, and the rule's weights times e^{lnL(x* + xi sigma)} are
// sigma W_i e^{K^2 / 2R}, so
//   ln L_d = K^2 / 2R + ln sigma + ln sum_i W_i p_x(x* + xi_i sigma),
//   p_x(x) = d_ref^3 x^-4 3 / (d_max^3 - d_min^3) on [d_ref/d_max, d_ref/d_min].
// No node inside the prior gives -inf; a poisoned sample gives NaN.  R >= 0
// holds exactly, so R <= 0 comes only from rounding where the model has no
// power (F_k Y = 0, hence K = 0 too): lnL = 0 at every distance and the
// marginal is the prior's mass, ln L_d = 0.
__device__ __forceinline__ double dist_marginal(const DistRule& G, double d_ref, const Terms& t) {
  const double Kd = t.data, Rd = 2.0 * t.quad;
  if (t.bad || !(fabs(Kd) <= 1.0e300) || !(fabs(Rd) <= 1.0e300)) return __builtin_nan("");
  if (!(Rd > 0.0)) return 0.0;
  const double xs = Kd / Rd;
  const double sig = 1.0 / sqrt(Rd);
  const double xlo = d_ref / G.d_max, xhi = d_ref / G.d_min;
  double s = 0.0;
  for (int i = 0; i < G.n; ++i) {
    const double x = fma(G.xi[i], sig, xs);
    if (x >= xlo && x <= xhi) {
      const double r = d_ref / x;  // D at the node: p_x = D^4 / d_ref (normalised below)
      const double r2 = r * r;
      s = fma(G.w[i], r2 * r2, s);
    }
  }
  if (!(s > 0.0)) return -__builtin_inf();
  // p_x(x) = d_ref^3 x^-4 exp(ln_norm) = (d_ref / x)^4 exp(ln_norm) / d_ref
  return 0.5 * Kd * xs + log(sig) + G.ln_norm - log(d_ref) + log(s);
}

// The fixed-spacing rule over geocentric time (Eq. (ap:tfixed)): n (odd)
// times t0 + k h, composite Simpson weights, prior uniform over the window.
struct TimeRule {
  int32_t n;
  int32_t pad;
  double t0, h;
  double ln_scale;                // ln(h / T) = -ln(n - 1), T = (n - 1) h
  double lw_end, lw_odd, lw_even;  // ln(1/3), ln(4/3), ln(2/3)
};

// ln of the likelihood marginalised over geocentric time, per sample:
//   ln L_t = ln[(h / T) sum_k w_k e^{lnL(t0 + k h)}].
// The model-norm term does not depend on time, so it is evaluated once; the
// data term once per time (new stencils, the same F and Y).  The log-sum
// runs online with one exp per time.  A poisoned sample gives NaN.  The
// whole wavefront calls this together (the data term reads cooperatively).
template <class R, int KT, int L>
__device__ __forceinline__ double eval_tmarg(PDesc P, R* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                             double ra, double dec, double psi, double incl, double phi, double dist,
                                             const TimeRule& T) {
  static_assert(sizeof(R) == 8, "FP64");
  reduce_angles<R>(psi, incl, phi);
  Sky<R, KT> S;
  R si, ci, sf, cf;
  sky_eval<R, KT, false>(P, ra, dec, psi, incl, phi, 0.0, S, si, ci, sf, cf);
  double wq = 0.0;
  const double quad = quad_term<R, KT, L, false>(P, trig, ts, ci, si, cf, sf, S.Fre, S.Fim, &wq);
  const double x = P->d_ref / dist;
  const double base = -x * x * quad;
  double m = -__builtin_inf(), sum = 0.0;
  bool bad = !(fabs(x) <= 1.0e300) || !(fabs(base) <= 1.0e300);
  for (int k = 0; k < T.n; ++k) {
    S.bad = false;
    sky_stencils<R, KT>(P, fma((double)k, T.h, T.t0), S);
    bad = bad || S.bad;
    const double data = data_norm<KT, L, false, false>(P, trig, ts, stage, S.row, S.sfr, S.Fre, S.Fim, ci, si, cf, sf,
                                                       nullptr, nullptr);
    const double lw = (k == 0 || k == T.n - 1) ? T.lw_end : ((k & 1) ? T.lw_odd : T.lw_even);
    const double l = fma(x, data, base) + lw;
    if (l > m) {
      sum = (sum == 0.0) ? 1.0 : fma(sum, exp(m - l), 1.0);
      m = l;
    } else {
      sum += exp(l - m);
    }
  }
  if (bad || !(m == m)) return __builtin_nan("");
  return m + log(sum) + T.ln_scale;
}

// The data pass of the band-limited full-window rule (Eq. (ap:tband)): at
// fixed other parameters the exponent is x kappa(t) - x^2 quad with kappa the
// band-limited data term; this pass takes x kappa at the T.n nodes
// t0 + k h (new stencils, the same F and Y) into kap[k N + i] (when `live`)
// and returns the time-independent -x^2 quad (NaN for a poisoned sample).
// The reconstruction between the nodes and the exponential sum run in a
// separate kernel over these values.  The whole wavefront calls this
// together (the data term reads cooperatively).
template <class R, int KT, int L>
__device__ __forceinline__ double eval_tkappa(PDesc P, R* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                              double ra, double dec, double psi, double incl, double phi, double dist,
                                              const TimeRule& T, RIFT_GLOBAL double* kap, int64_t N, int64_t i,
                                              bool live) {
  static_assert(sizeof(R) == 8, "FP64");
  reduce_angles<R>(psi, incl, phi);
  Sky<R, KT> S;
  R si, ci, sf, cf;
  sky_eval<R, KT, false>(P, ra, dec, psi, incl, phi, 0.0, S, si, ci, sf, cf);
  double wq = 0.0;
  const double quad = quad_term<R, KT, L, false>(P, trig, ts, ci, si, cf, sf, S.Fre, S.Fim, &wq);
  const double x = P->d_ref / dist;
  const double base = -x * x * quad;
  bool bad = !(fabs(x) <= 1.0e300) || !(fabs(base) <= 1.0e300);
  for (int k = 0; k < T.n; ++k) {
    S.bad = false;
    sky_stencils<R, KT>(P, fma((double)k, T.h, T.t0), S);
    bad = bad || S.bad;
    const double data = data_norm<KT, L, false, false>(P, trig, ts, stage, S.row, S.sfr, S.Fre, S.Fim, ci, si, cf, sf,
                                                       nullptr, nullptr);
    if (live) kap[(int64_t)k * N + i] = x * data;
  }
  return bad ? __builtin_nan("") : base;
}

// The data pass of the polarisation marginal: at fixed other parameters lnL is
//   q(u) = a + Re(c1 e^{iu}) + Re(c2 e^{2iu}),  u = 2 (psi' - psi)
// (Eq. (ap:psiexp)).  With the data term as the complex W = sum_k conj(F_k) Z_k
// (one gather), the model-norm term as A0 = sum_k |F_k|^2 a_k / 4 and
// B = sum_k F_k^2 b_k / 4 (one contraction), and F_k(psi + u/2) = e^{-iu} F_k(psi),
//   q(u) = x Re(e^{iu} W) - x^2 [A0 + Re(e^{-2iu} B)]:
//   a = -x^2 A0, c1 = x W, c2 = -x^2 conj(B),
// into out rows (a, Re c1, Im c1, Re c2, Im c2) of stride N (when `live`).
// Returns whether the sample is poisoned.  The rules over u run in a kernel of
// their own over these five values.
constexpr int PSI_ROWS = 5;
template <class R, int KT, int L>
__device__ __forceinline__ bool eval_pmarg(PDesc P, R* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                           double ra, double dec, double psi, double incl, double phi, double tref,
                                           double dist, RIFT_GLOBAL double* out, int64_t N, int64_t i, bool live) {
  reduce_angles<R>(psi, incl, phi);
  Sky<R, KT> S;
  R si, ci, sf, cf;
  sky_eval<R, KT, true>(P, ra, dec, psi, incl, phi, tref, S, si, ci, sf, cf);
  static_assert(sizeof(R) == 8, "FP64");
  double wim = 0.0;
  R acc[3 * KT];
  const double wre = data_norm<KT, L, true, true>(P, trig, ts, stage, S.row, S.sfr, S.Fre, S.Fim, ci, si, cf, sf, acc,
                                                  &wim);
  double A0 = 0.0, Bre = 0.0, Bim = 0.0;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const R f2 = S.Fre[k] * S.Fre[k] + S.Fim[k] * S.Fim[k];
    const R g2r = S.Fre[k] * S.Fre[k] - S.Fim[k] * S.Fim[k];
    const R g2i = 2 * S.Fre[k] * S.Fim[k];
    A0 += (double)(f2 * acc[3 * k]);
    Bre += (double)(g2r * acc[3 * k + 1]) + (double)(g2i * acc[3 * k + 2]);
    Bim += (double)(g2i * acc[3 * k + 1]) - (double)(g2r * acc[3 * k + 2]);
  }
  const double x = P->d_ref / dist;
  const double x2 = x * x;
  if (live) {
    out[i] = -x2 * A0;
    out[N + i] = x * wre;
    out[2 * N + i] = x * wim;
    out[3 * N + i] = -x2 * Bre;
    out[4 * N + i] = x2 * Bim;
  }
  return S.bad || !(fabs(x) <= 1.0e300) || !(fabs(wre) <= 1.0e300) || !(fabs(wim) <= 1.0e300) ||
         !(fabs(A0) <= 1.0e300) || !(fabs(Bre) + fabs(Bim) <= 1.0e300);
}

// The data pass of the joint phiref / psi marginal by exact reconstruction
// (ERAI, Eqs. (ap:angleharm), (ap:nyquist)).  At fixed sky, inclination,
// time and distance, lnL in the offsets (alpha of phiref, u = 2 (psi' - psi)) is
//   q(alpha, u) = a(alpha) + Re(c1(alpha) e^{iu}) + Re(c2(alpha) e^{2iu}),
// c1 = x W (the complex data term), a = -x^2 A0 and c2 = -x^2 conj(B) (the model
// norm), as in the polarisation marginal.  In alpha, c1 is a trigonometric
// polynomial of degree m_max and a, c2 of degree 2 m_max, and their
// coefficients come out of one evaluation:
//   W(alpha) = sum_m T_m e^{-i m alpha}, T_m = e^{-i m phi} sum_k conj(F_k) sum_{i: m_i = m} d_i Qhat_{k,i},
// the sums of one gather kept apart by m, and the model norm's basis rows kept
// apart by q.  (Sampling q at 2 m_max + 1 data-term and 4 m_max + 1 model-norm
// phases took nine gathers and seventeen contractions at m_max = 4: 2.5 ms for
// 1e6 samples at 3 detectors and 21 modes, now 0.7 ms.)
//   out rows [2 j], [2 j + 1], j < nd = 2 m_max + 1: Re, Im c1 along 1, cos alpha,
//   sin alpha, .., sin m_max alpha; rows [2 nd + 3 j + 0 .. 2], j < nq = 4 m_max + 1:
//   a, Re c2, Im c2 along 1, cos alpha, .., sin 2 m_max alpha; stride N (when `live`).
// Returns whether the sample is poisoned.  The whole wavefront calls this together.
struct AngleRule {
  int32_t nd, nq;
};
constexpr int ERAI_MAX_M = 4;

// T[m + ERAI_MAX_M] += sum_k conj(F_k) sum_{i: m_i = m} d_i Qhat_{k,i}.
template <int KT, int L, int W>
__device__ __forceinline__ void data_harmonics_w(PDesc P, RIFT_LDS unsigned char* stage, const int32_t* row,
                                               const double* sfr, const double* Fre, const double* Fim, double ci,
                                               double si, C2<double>* T) {
  const int M = P->M, rows = P->n_t + 2 * QPAD;
  double d[W], qx[W], qy[W];
  int m[W];
  RowReader<KT, W> R;
  ModeWalk<L + 1> mode;
#pragma unroll 1
  for (int window = 0; window < rows; window += ROWS_WINDOW) {
    R.start(P, stage, row, window);
#pragma unroll 1
    while (R.left > 0) {
      double w[4];
      lagrange4(by_det<KT>(sfr, R.k), w);
#pragma unroll
      for (int t = 0; t < RowReader<KT, W>::UNITS; ++t) {
        R.ahead(t);
        if (R.k == 0) {
          mode.fetch(P, R.p * W + 2 * t, M);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            m[2 * t + j] = uniform_i(mode.m[j]);
            d[2 * t + j] = mode.d(j, ci, si);
          }
        }
        Cplx v[8];
        R.fetch(t, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int r = t * (8 / W) + c / W, s = c % W;
          qx[s] = r == 0 ? w[r] * v[c].x : fma(w[r], v[c].x, qx[s]);
          qy[s] = r == 0 ? w[r] * v[c].y : fma(w[r], v[c].y, qy[s]);
          pin(qx[s]);
          pin(qy[s]);
        }
      }
      const double fr = by_det<KT>(Fre, R.k), fi = by_det<KT>(Fim, R.k);
      const bool in = rows <= ROWS_WINDOW || in_window(by_det<KT>(row, R.k), window);
      // the modes are sorted by m: the running sum goes to T where m changes
      double zr = 0.0, zi = 0.0;
#pragma unroll
      for (int s = 0; s < W; ++s) {
        zr = fma(d[s], qx[s], zr);
        zi = fma(d[s], qy[s], zi);
        if (s + 1 == W || m[s + 1] != m[s]) {
          if (!in) zr = zi = 0.0;
          const double tr = fma(fr, zr, fi * zi), ti = fma(fr, zi, -fi * zr);
#pragma unroll
          for (int j = 0; j < 2 * ERAI_MAX_M + 1; ++j) {
            if (j == m[s] + ERAI_MAX_M) {  // uniform
              T[j].x += tr;
              T[j].y += ti;
            }
          }
          zr = zi = 0.0;
        }
      }
#pragma unroll
      for (int j = 0; j < 2 * ERAI_MAX_M + 1; ++j) {
        pin(T[j].x);
        pin(T[j].y);
      }
      R.advance();
    }
  }
}

template <int KT, int L>
__device__ __forceinline__ void data_harmonics(PDesc P, RIFT_LDS unsigned char* stage, const int32_t* row,
                                               const double* sfr, const double* Fre, const double* Fim, double ci,
                                               double si, C2<double>* T) {
  if constexpr (Cls<L>::MAXM > QW64_SHORT_MODES) {
    if (P->w64 == QW64) {
      data_harmonics_w<KT, L, QW64>(P, stage, row, sfr, Fre, Fim, ci, si, T);
      return;
    }
  }
  data_harmonics_w<KT, L, QW64_SHORT>(P, stage, row, sfr, Fre, Fim, ci, si, T);
}

// The model norm's harmonics in alpha: for every q, the basis rows' sums over
// the degrees in incl along cos(q phi) and sin(q phi) for all 3 KT columns,
// combined with the detectors' F and turned by q phi.  The coefficients
// stream as in Contract; `emit(q, s, A, Br, Bi)` takes the parts along
// cos q alpha (s = 0) and sin q alpha (s = 1) of A0, Re B and Im B.
template <int KT, int L>
struct NormHarmonics {
  static constexpr int NI = 2 * L, W = 3 * KT, B = Cls<L>::B;
  static constexpr int NC = B * W, CH = 16, NCH = (NC + CH - 1) / CH;
  struct State {
    double ct[NI + 1], st[NI + 1];  // cos(n incl), sin(n incl)
    double pc[W], ps[W];            // the sums of the current q
    double ex, ey;                  // e^{i q phi}
  };
  template <int C>
  static __device__ __forceinline__ void ld(double (&buf)[CH], const RIFT_CONST double* Cc) {
    const RIFT_CONST double* p = opaque(Cc) + C * CH;
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (C * CH + i < NC) buf[i] = p[i];
  }
  template <class Emit>
  static __device__ __forceinline__ void close(int q, const double* Fre, const double* Fim, State& S, Emit&& emit) {
    double v[2][3];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const double* p = s ? S.ps : S.pc;
      double A = 0.0, Br = 0.0, Bi = 0.0;
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        const double f2 = Fre[k] * Fre[k] + Fim[k] * Fim[k];
        const double gr = Fre[k] * Fre[k] - Fim[k] * Fim[k], gi = 2 * Fre[k] * Fim[k];
        A = fma(f2, p[3 * k], A);
        Br = fma(gr, p[3 * k + 1], fma(gi, p[3 * k + 2], Br));
        Bi = fma(gi, p[3 * k + 1], fma(-gr, p[3 * k + 2], Bi));
      }
      v[s][0] = A;
      v[s][1] = Br;
      v[s][2] = Bi;
    }
    // cos q (phi + alpha), sin q (phi + alpha) along cos q alpha, sin q alpha
    emit(q, 0, fma(v[0][0], S.ex, v[1][0] * S.ey), fma(v[0][1], S.ex, v[1][1] * S.ey),
         fma(v[0][2], S.ex, v[1][2] * S.ey));
    if (q > 0)
      emit(q, 1, fma(v[1][0], S.ex, -v[0][0] * S.ey), fma(v[1][1], S.ex, -v[0][1] * S.ey),
           fma(v[1][2], S.ex, -v[0][2] * S.ey));
#pragma unroll
    for (int c = 0; c < W; ++c) S.pc[c] = S.ps[c] = 0.0;
  }
  template <int J, class Emit>
  static __device__ __forceinline__ void coef(double c, double cf, double sf, const double* Fre, const double* Fim,
                                              State& S, Emit&& emit) {
    if constexpr (J < NC) {
      constexpr int b = J / W, col = J % W, rb = basis_row<L>(b);
      constexpr int kind = rb & 15, n = (rb >> 4) & 255, q = rb >> 12;
      const double t = kind >= 3 ? S.st[n] : S.ct[n];
      double& p = (kind == 2 || kind == 4) ? S.ps[col] : S.pc[col];
      p = fma(c, t, p);
      if constexpr (col == W - 1 && (b + 1 == B || (basis_row<L>(b + 1) >> 12) != q)) {
        close(q, Fre, Fim, S, emit);
        phase_up_to(S, cf, sf);
      }
    }
  }
  static __device__ __forceinline__ void phase_up_to(State& S, double cf, double sf) {
    const double a = S.ex * cf - S.ey * sf, b = S.ex * sf + S.ey * cf;
    S.ex = a;
    S.ey = b;
  }
  template <int C, class Emit, int... I>
  static __device__ __forceinline__ void fm(const double (&buf)[CH], double cf, double sf, const double* Fre,
                                            const double* Fim, State& S, Emit&& emit, std::integer_sequence<int, I...>) {
    (coef<C * CH + I>(buf[I], cf, sf, Fre, Fim, S, emit), ...);
  }
  template <int C, class Emit>
  static __device__ __forceinline__ void step(const RIFT_CONST double* Cc, double (&cur)[CH], double (&nxt)[CH],
                                              double cf, double sf, const double* Fre, const double* Fim, State& S,
                                              Emit&& emit) {
    if constexpr (C < NCH) {
#pragma unroll
      for (int i = 0; i < CH; ++i)
        if (C * CH + i < NC) pin_s(cur[i]);
      if constexpr (C + 1 < NCH) ld<C + 1>(nxt, Cc);
      fm<C>(cur, cf, sf, Fre, Fim, S, emit, std::make_integer_sequence<int, CH>{});
#pragma unroll
      for (int c = 0; c < W; ++c) {
        pin(S.pc[c]);
        pin(S.ps[c]);
      }
      step<C + 1>(Cc, nxt, cur, cf, sf, Fre, Fim, S, emit);
    }
  }
  template <class Emit>
  static __device__ __forceinline__ void run(PDesc P, double* __restrict__ trig, int ts, double ci, double si,
                                             double cf, double sf, const double* Fre, const double* Fim, Emit&& emit) {
    State S;
    S.ex = 1.0;
    S.ey = 0.0;
#pragma unroll
    for (int c = 0; c < W; ++c) S.pc[c] = S.ps[c] = 0.0;
    const RIFT_CONST double* Cc = as_const(P->C64);
    if constexpr (L <= 4) {
      S.ct[0] = 1.0;
      S.st[0] = 0.0;
      S.ct[1] = ci;
      S.st[1] = si;
#pragma unroll
      for (int n = 2; n <= NI; ++n) {
        S.ct[n] = 2.0 * ci * S.ct[n - 1] - S.ct[n - 2];
        S.st[n] = 2.0 * ci * S.st[n - 1] - S.st[n - 2];
      }
      double bA[CH], bB[CH];
      ld<0>(bA, Cc);
      step<0>(Cc, bA, bB, cf, sf, Fre, Fim, S, emit);
    } else {
      // runtime rows; cos, sin(n incl) in this lane's column of the scratch
      double c0 = 1.0, c1 = ci, s0 = 0.0, s1 = si;
#pragma unroll
      for (int n = 0; n <= NI; ++n) {
        trig[n * ts] = n == 0 ? c0 : c1;
        trig[(NI + 1 + n) * ts] = n == 0 ? s0 : s1;
        if (n > 0) {
          const double c2 = 2.0 * ci * c1 - c0, s2 = 2.0 * ci * s1 - s0;
          c0 = c1;
          c1 = c2;
          s0 = s1;
          s1 = s2;
        }
      }
      int b = 0;
#pragma unroll 1
      for (int q = 0; q <= 4 * ERAI_MAX_M / 2; ++q) {  // the rows of higher q are zero for |m| <= ERAI_MAX_M
        const int odd = q & 1, base = odd ? NI + 1 : 0;
#pragma unroll 1
        for (int n = odd; n <= NI; ++n) {
          const double t = trig[(base + n) * ts];
#pragma unroll
          for (int c = 0; c < W; ++c) S.pc[c] = fma(Cc[b * W + c], t, S.pc[c]);
          ++b;
          if (q > 0) {
#pragma unroll
            for (int c = 0; c < W; ++c) S.ps[c] = fma(Cc[b * W + c], t, S.ps[c]);
            ++b;
          }
        }
        close(q, Fre, Fim, S, emit);
        phase_up_to(S, cf, sf);
      }
    }
  }
};

template <int KT, int L>
__device__ __forceinline__ bool eval_erai(PDesc P, double* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                          double ra, double dec, double psi, double incl, double phi, double tref,
                                          double dist, const AngleRule& R, RIFT_GLOBAL double* out, int64_t N,
                                          int64_t i, bool live) {
  Sky<double, KT> S;
  double si, ci, sf, cf;
  sky_eval<double, KT, true>(P, ra, dec, psi, incl, phi, tref, S, si, ci, sf, cf);
  const double x = P->d_ref / dist;
  const double x2 = x * x;
  C2<double> T[2 * ERAI_MAX_M + 1];
#pragma unroll
  for (int j = 0; j < 2 * ERAI_MAX_M + 1; ++j) T[j].x = T[j].y = 0.0;
  __builtin_amdgcn_s_setprio(1);
  data_harmonics<KT, L>(P, stage, S.row, S.sfr, S.Fre, S.Fim, ci, si, T);
  __builtin_amdgcn_s_setprio(0);
  bool bad = S.bad || !(fabs(x) <= 1.0e300);
  // x T_m e^{-i m phi}, then c1 along 1, cos m alpha, sin m alpha
  const int mm = (R.nd - 1) / 2;
  {
    double ex = 1.0, ey = 0.0;
#pragma unroll
    for (int m = 0; m <= ERAI_MAX_M; ++m) {
      const C2<double> p = T[ERAI_MAX_M + m], n = T[ERAI_MAX_M - m];
      // T_m e^{-i m phi} and T_-m e^{i m phi}
      const double pr = x * (p.x * ex + p.y * ey), pi = x * (p.y * ex - p.x * ey);
      const double nr = x * (n.x * ex - n.y * ey), ni = x * (n.y * ex + n.x * ey);
      bad = bad || !(fabs(pr) + fabs(pi) + fabs(nr) + fabs(ni) <= 1.0e300);
      if (live && m <= mm) {
        if (m == 0) {
          out[i] = pr;
          out[N + i] = pi;
        } else {
          RIFT_GLOBAL double* o = out + (int64_t)(2 * (2 * m - 1)) * N + i;
          o[0] = pr + nr;
          o[N] = pi + ni;
          o[2 * N] = pi - ni;
          o[3 * N] = nr - pr;
        }
      }
      const double a = ex * cf - ey * sf, b = ex * sf + ey * cf;
      ex = a;
      ey = b;
    }
  }
  const int r0 = 2 * R.nd;
  NormHarmonics<KT, L>::run(P, trig, ts, ci, si, cf, sf, S.Fre, S.Fim,
                            [&](int q, int s, double A, double Br, double Bi) {
                              bad = bad || !(fabs(A) <= 1.0e300) || !(fabs(Br) + fabs(Bi) <= 1.0e300);
                              if (live && q <= 2 * mm) {
                                RIFT_GLOBAL double* o =
                                    out + (int64_t)(r0 + 3 * (q == 0 ? 0 : 2 * q - 1 + s)) * N + i;
                                o[0] = -x2 * A;
                                o[N] = -x2 * Br;
                                o[2 * N] = x2 * Bi;
                              }
                            });
  // this class's degrees end at 2 L; another point of the plan may have more
  for (int r = r0 + 3 * (4 * L + 1); live && r < r0 + 3 * R.nq; ++r) out[(int64_t)r * N + i] = 0.0;
  return bad;
}

// Everything per sample up to the distance: the terms.  R is the arithmetic
// type of the bulk (FP64 or FP32); the sky frame, delays and the final
// combination are always FP64.  `stage` is this wavefront's STAGE_WAVE bytes of
// LDS; the whole wavefront must call these together.
template <class R, int KT, int L, bool BOUND>
__device__ __forceinline__ Terms eval_terms(PDesc P, R* __restrict__ trig, int ts, RIFT_LDS unsigned char* stage,
                                            double ra, double dec, double psi, double incl, double phi,
                                            double tref) {
  reduce_angles<R>(psi, incl, phi);
  Sky<R, KT> S;
  R si, ci, sf, cf;
  sky_eval<R, KT, true>(P, ra, dec, psi, incl, phi, tref, S, si, ci, sf, cf);
  Terms t;
  t.wq = 0.0;
  if constexpr (sizeof(R) == 8) {
    static_assert(!BOUND, "the bound is the FP32 pass's");
    double acc[3 * KT];
    t.data = data_norm<KT, L, true, false>(P, trig, ts, stage, S.row, S.sfr, S.Fre, S.Fim, ci, si, cf, sf, acc, nullptr);
    t.quad = quad_of<double, KT, false>(P, acc, S.Fre, S.Fim, &t.wq);
  } else {
    constexpr int NY = Cls<L>::NY;
    R cn[NY], sn[NY];
    incl_harmonics<R, NY>(ci, si, cn, sn);
    __builtin_amdgcn_s_setprio(1);
    t.data = data_direct<R, KT, L>(P, stage, S.row, S.sfr, S.Fre, S.Fim, cn, sn, cf, sf);
    __builtin_amdgcn_s_setprio(0);
    t.quad = quad_term<R, KT, L, BOUND>(P, trig, ts, ci, si, cf, sf, S.Fre, S.Fim, &t.wq);
  }
  t.bad = S.bad;
  return t;
}

template <class R, int KT, int L, bool BOUND>
__device__ __forceinline__ Eval eval_sample(PDesc P, R* __restrict__ trig, int ts,
                                            RIFT_LDS unsigned char* stage, double ra, double dec, double psi,
                                            double incl, double phi, double tref, double dist) {
  const Terms t = eval_terms<R, KT, L, BOUND>(P, trig, ts, stage, ra, dec, psi, incl, phi, tref);
  return combine<BOUND>(P, dist, t.data, t.quad, t.wq, t.bad);
}

// ---------------------------------------------------------------------------
// log-sum-exp pairs (max, sum exp(l - max)); NaN propagates through the sum.
// ---------------------------------------------------------------------------
struct MS {
  double m, s;
};
__device__ __forceinline__ MS ms_of(double l) {
  MS r;
  if (l != l) {
    r.m = -__builtin_inf();
    r.s = __builtin_nan("");
  } else if (l == -__builtin_inf()) {
    r.m = l;
    r.s = 0.0;
  } else {
    r.m = l;
    r.s = 1.0;
  }
  return r;
}
// Add one sample's l to (max, sum): one exp instead of two.
__device__ __forceinline__ MS ms_push(MS a, double l) {
  if (l != l) {  // NaN poisons the sum
    a.s = __builtin_nan("");
    return a;
  }
  if (l == -__builtin_inf()) return a;
  if (l > a.m) {
    a.s = (a.s == 0.0) ? 1.0 : a.s * exp(a.m - l) + 1.0;
    a.m = l;
  } else {
    a.s += exp(l - a.m);
  }
  return a;
}
__device__ __forceinline__ MS ms_combine(MS a, MS b) {
  MS r;
  r.m = fmax(a.m, b.m);
  const double ta = (a.s == 0.0) ? 0.0 : a.s * exp(a.m - r.m);
  const double tb = (b.s == 0.0) ? 0.0 : b.s * exp(b.m - r.m);
  r.s = ta + tb;
  return r;
}
__device__ __forceinline__ MS ms_wave(MS v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    MS o;
    o.m = __shfl_xor(v.m, off);
    o.s = __shfl_xor(v.s, off);
    v = ms_combine(v, o);
  }
  return v;
}
// Block-wide reduction in a fixed order (deterministic).  `sh` holds one MS
// per wave.
__device__ __forceinline__ MS ms_block(MS v, MS* sh) {
  v = ms_wave(v);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  MS r = sh[0];
  for (int w = 1; w < nw; ++w) r = ms_combine(r, sh[w]);
  return r;
}

__device__ __forceinline__ double dmax_wave(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ double dsum_wave(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

}  // namespace rift
