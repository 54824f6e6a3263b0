// The composite-index likelihood of the generalised detector response
// (Sec. "A generalized detector response"): the mode index widens to
// A = (a, lm) and the static antenna factor F_k to a coefficient C~^k_a per
// composite term a, Eq. (slowrot:lnL:Decomposed):
//
//   lnL = x Re sum_k sum_a sum_lm conj(C~^k_a Y_lm) Q_{k,a lm}(t_k)
//       - x^2/4 sum_k [ c_k^H U_k c_k + Re(c_k^T V_k c_k) ],   c_{k,(a,lm)} = C~^k_a Y_lm.
//
// Two responses:
//   rotation (Path A): a <-> sidereal harmonic n = a - 2, n = -2..2.  F_k over
//     the Greenwich hour angle g is a degree-2 trigonometric polynomial,
//     F_k(g) = sum_n A_n e^{i n g} (Eq. (slowrot:Fharm)); A_n in closed form
//     of the sample's dec and psi.
//     C~_n = A_n e^{i n g(t_ref)} e^{i n W (t_k - t_ref)} (the post-phase
//     of Eq. (slowrot:postphase), the bank's modulation referenced to the
//     template's own time), g(t) = gmst + W t - ra; the delay is held at the
//     arrival time t_k of the sky frame at t_ref.
//   arms (Path D): a <-> order p of the arm-projection expansion,
//     b_p = 1/2 [ (x.N)^p e:xx - (y.N)^p e:yy ] (Eq. (fsize:bp)) with
//     e:aa = (X.a + i Y.a)^2 for the complex polarisation tensor e = e+ + i ex;
//     static sky frame.
//
// A wavefront evaluates 64 samples, in FP64.  The front (sky frame, harmonics,
// coefficients) and the data term take a lane per sample.
//
// The quadratic term is one real form.  With c_a = C~_a Y as real values,
//   Re(c_a^H U_ab c_b) + Re(c_a^T V_ab c_b) = c_a^T S_ab c_b,
//   S(i, j) = [ Ur + Vr   -Ui - Vi ]
//             [ Ui - Vi    Ur - Vr ]  of the modes' entry (i, j),
// summed over a <= b, off the diagonal twice (U Hermitian, V symmetric): a
// quarter of the multiply-adds of the two complex forms over all pairs.  For
// the 64 samples of a wavefront, S c is a dense product with one matrix for
// all of them, so it runs on the FP64 matrix cores (16 x 16 x 4 tiles): the
// matrix streams past as A operands in whole lines, each used for 64 samples,
// with the values c as B operands in four tiles of 16 samples.  (On the vector
// unit the matrix had to reach the lanes as scalar operands, and their
// latency, not the multiply-adds, set the time: up to 3000 dependent scalar
// loads a wavefront for the composite forms, with two wavefronts a SIMD.)
// Measured (3 detectors, 6554-row windows, a call; the forms on the vector unit
// before): rotation, 4 modes, 1e6 samples 724 -> 374 us; 9 modes, 1000 and 150k
// samples 689 -> 131 and 1235 -> 354 us; 21 modes, 20k and 200k samples
// 588 -> 354 and 1155 -> 1128 us; 12 terms (the drift to order 1), 4 modes, 1e6
// samples 3.6 -> 1.47 ms.  At 1e6 samples of the rotation the rows of Q alone take
// 0.15 ms to read, the matrix products 0.09 and the front about 0.13: a second
// pair of wavefronts a SIMD (staging halved to make the LDS for it) or products
// issued between the lines of Q, both of which spill, gave no more.
//
// The complete l <= 4 set of 21 modes also has the form per pair of terms in the
// static path's harmonic basis, which needs fewer operations (wide_harmonic).
//
// The data term reads Q by rows: a set-up kernel lays every detector's
// composite entries of one time out as whole 128-byte lines.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/rift_ile.h"
#include "ile_device.h"
#include "ile_host.h"

namespace rift {
namespace {

constexpr int WIDE_ARMS_MAX_TERMS = 8;
constexpr int WIDE_MERGE = 1024;      // threads of the merge
constexpr int WIDE_BASIS_BLOCK = 512;  // threads of the harmonic set-up: one per grid point

struct WideDesc {
  int32_t K, M, n_t, n_a, response;
  int32_t npairs;            // pairs of terms a <= b
  double t0, inv_dt, gmst, omega, d_ref;
  double dten[KMAX][6];      // D00, D11, D22, 2 D01, 2 D02, 2 D12
  double rpos[KMAX][3];      // light-seconds
  double arms[KMAX][2][3];   // arm unit vectors
  int32_t perm[MMAX];        // caller's index of internal mode i (modes sorted by m)
  int32_t m[MMAX];
  int32_t odd[MMAX];
  double ycoef[MMAX][LMAXC + 1];
  const double* Q;           // caller's [K][n_a][M][n_t] complex
  const double* Qrows;       // the same by rows (k_wide_rows), where the call repacks it
  const double* S;           // the real form's operands (k_wide_form), or [K][pair][B][4] (k_wide_basis)
};
static_assert(sizeof(WideDesc) <= 3584, "the description travels as a kernel argument");

// Polarisation axes X, Y at hour angle g for dec, psi (the static sky frame).
__device__ __forceinline__ void axes(double sg, double cg, double sd, double cd, double sp, double cp, double* X,
                                     double* Y, double* N) {
  const double ea[3] = {sg, cg, 0.0};
  const double ed[3] = {-sd * cg, sd * sg, cd};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    X[i] = -cp * ea[i] + sp * ed[i];
    Y[i] = sp * ea[i] + cp * ed[i];
  }
  N[0] = cd * cg;
  N[1] = -cd * sg;
  N[2] = sd;
}

// The composite values c_{a,m} = C~_a Y_m of one sample as real components in
// steps of four: step b = 2 (a MB + mb) + part holds the part (0 real, 1
// imaginary) of modes m = 4 mb + q at quad q = 0..3.  A tile is four steps
// (16 components); a form's product with tile t as rows takes the steps from
// the tile's own on.
__host__ __device__ constexpr int wide_steps(int MB, int n_a) { return 2 * MB * n_a; }
__host__ __device__ constexpr int wide_tiles(int MB, int n_a) { return (wide_steps(MB, n_a) + 3) / 4; }
// Pairs of steps (both parts of four modes of a term) that tiles 0 .. t-1 take.
__host__ __device__ constexpr int64_t wide_pairs(int steps, int t) { return (int64_t)t * (steps / 2) - (int64_t)t * (t - 1); }

// The A operands of every detector, [k][tile][pair of steps][lane][2]: lane l
// holds, for both steps b of the pair, the coefficient of row component
// (step 4 t + (l & 15) / 4, quad l & 3) and column component (step b, quad
// l >> 4): S summed over both orders of the two components where the column
// lies beyond the row's tile, S itself inside the tile (whose rows and columns
// meet in both orders).
template <int MB>
__global__ void k_wide_form(WideDesc D, const double* __restrict__ U, const double* __restrict__ V,
                            double* __restrict__ out) {
  const int steps = wide_steps(MB, D.n_a), tiles = wide_tiles(MB, D.n_a);
  const int64_t per_det = wide_pairs(steps, tiles) * 128;
  const int A = D.n_a * D.M;
  auto entry = [&](int k, int bi, int qi, int bj, int qj) {
    const int ai = bi / (2 * MB), aj = bj / (2 * MB);
    const int mi = 4 * ((bi % (2 * MB)) / 2) + qi, mj = 4 * ((bj % (2 * MB)) / 2) + qj;
    if (ai > aj || aj >= D.n_a || mi >= D.M || mj >= D.M) return 0.0;
    const int64_t o = 2 * (((int64_t)k * A + ai * D.M + D.perm[mi]) * A + aj * D.M + D.perm[mj]);
    const double f = ai == aj ? 1.0 : 2.0;
    const int pi = bi & 1, pj = bj & 1;
    if (pi == pj) return f * (pi ? U[o] - V[o] : U[o] + V[o]);
    return f * (pi ? U[o + 1] - V[o + 1] : -U[o + 1] - V[o + 1]);
  };
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < D.K * per_det;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(x / per_det);
    const int64_t r = x - k * per_det;
    const int e = (int)(r & 1), l = (int)((r >> 1) & 63);
    const int64_t pr = r >> 7;
    int t = 0;
    while (t + 1 < tiles && wide_pairs(steps, t + 1) <= pr) ++t;
    const int b = 4 * t + 2 * (int)(pr - wide_pairs(steps, t)) + e;
    const int bi = 4 * t + ((l & 15) >> 2), qi = l & 3, qj = l >> 4;
    double v = 0.0;
    if (bi < steps) {
      v = entry(k, bi, qi, b, qj);
      if (b >= 4 * t + 4) v += entry(k, b, qj, bi, qi);
    }
    out[x] = v;
  }
}

// Slots of one term in a row of the repacked table (a multiple of eight, or
// four for up to four modes), and the 128-byte lines (eight slots) of a row.
__host__ __device__ constexpr int wide_slots(int MB) { return MB == 1 ? 4 : 8 * ((MB + 1) / 2); }
__host__ __device__ constexpr int wide_lines(int MB, int n_a) { return (n_a * wide_slots(MB) + 7) / 8; }

// Q [K][n_a][M][n_t] -> [K][n_t][lines of eight slots]: every row of a
// detector's window is whole, aligned 128-byte lines holding all composite
// entries (term a, internal mode m) at slot a SL + m, zero where there is
// none.  A 64-row tile goes through LDS: series are read and rows written in
// whole lines.
constexpr int WIDE_QT = 64;
__global__ void __launch_bounds__(256) k_wide_rows(WideDesc D, int SL, int lines, double* __restrict__ out) {
  constexpr int CH = 8;  // one line of slots at a time
  __shared__ double2 tile[WIDE_QT][CH + 1];
  const int k = blockIdx.y, t0 = blockIdx.x * WIDE_QT;
  const double* Q = D.Q + 2 * (int64_t)k * D.n_a * D.M * D.n_t;
  double2* o = reinterpret_cast<double2*>(out) + (int64_t)k * D.n_t * lines * 8;
  for (int l = blockIdx.z; l < lines; l += gridDim.z) {
    for (int x = threadIdx.x; x < CH * WIDE_QT; x += blockDim.x) {
      const int sl = x / WIDE_QT, t = x - (x / WIDE_QT) * WIDE_QT;
      const int e = l * 8 + sl, a = e / SL, m = e - (e / SL) * SL;
      double2 v = make_double2(0.0, 0.0);
      if (a < D.n_a && m < D.M && t0 + t < D.n_t) {
        const double* q = Q + 2 * (((int64_t)a * D.M + D.perm[m]) * D.n_t + t0 + t);
        v = make_double2(q[0], q[1]);
      }
      tile[t][sl] = v;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < CH * WIDE_QT; x += blockDim.x) {
      const int t = x / CH, sl = x - (x / CH) * CH;
      if (t0 + t < D.n_t) o[((int64_t)(t0 + t) * lines + l) * 8 + sl] = tile[t][sl];
    }
    __syncthreads();
  }
}

// Whether a call reads Q by rows.  Repacking costs a launch and a pass over the
// table (5 us at least), and its staging 12 KB of LDS a wavefront: from four terms
// on seven wavefronts fit a CU instead of the eight that its registers hold, from
// seven on fewer.  Measured (3 detectors, us, series as they are against rows):
//   up to a wavefront on every SIMD, bound by the latency of the reads: 21 modes x
//     5 terms 409, 366; 9 x 5 152, 143; 12 x 4 131, 112; 4 x 5 with 8 detectors
//     124, 108; but 4 x 5 51, 54; 16 x 3 143, 144; 8 x 8 175, 184;
//   more, bound by the lines that are read: 1e6 samples of 4 x 5 440, 370; 8 x 4
//     772, 585; 16 x 5 2508, 2160; 21 x 2 1266, 1045; 12 x 1 282, 242.  Rows of which
//     a quarter and more is empty read no fewer lines (4 x 1 131, 143; 2 x 5 311,
//     365; 5 x 5 755, 793), and many terms lose more by the LDS (4 x 8 720, 661, but
//     4 x 21 3355, 4388; 12 x 12 6085, 7617; 25 x 5 1662, 2082 at 262144).  Seven
//     wavefronts instead of eight count where they begin another round (16 x 5,
//     1e5 samples, one round each: 356, 306; 4 x 5, 131072: 76, 85; 2e5: 121, 108).
bool wide_packs(int K, int M, int n_a, int64_t n) {
  constexpr int64_t EIGHT = 131072, SEVEN = 114688;  // samples of a round on 256 CUs
  const int MB = (M + 3) / 4;
  if (n < 16384) return false;
  if (n <= EIGHT / 2) return M >= 9 ? n_a >= 4 && M * n_a >= 45 : M == 4 && n_a <= 12 && K * n_a >= 36;
  if (M < 4 || M > 24 || (M < 9 && 4 * M * n_a < 3 * 8 * wide_lines(MB, n_a))) return false;
  if (n_a <= 3) return n * M * n_a >= 2400000;
  if (n_a > 6) return M == 4 && n_a <= 8 && n >= 200000;
  if (n >= 400000) return n_a == 4 || M <= 16;
  return (n + SEVEN - 1) / SEVEN <= (n + EIGHT - 1) / EIGHT;
}

// A wavefront's coefficients C~ [term][lane].
typedef RIFT_LDS double2* WideCoef;

// Re sum_a conj(C~_a) sum_m conj(Y_m) Qhat_{a,m} of one detector from the
// repacked table: the stencil's four rows are 4 x lines aligned 128-byte lines
// per lane, read cooperatively through LDS as the static path reads its
// blocks (eight lanes fetch the eight 16-byte chunks of one lane's line,
// straight to LDS, two 8 KB buffers per wavefront; the same chunk swizzle).
// Rows jc .. jc + 3 at byte offset `boff` of detector k's table, tap weights
// wr.  The whole wavefront calls this together.
template <int MB>
__device__ __forceinline__ double wide_data(const RIFT_GLOBAL char* tab, uint32_t boff, int n_a,
                                            RIFT_LDS unsigned char* stage, const double* wr, const double* yr,
                                            const double* yi, WideCoef C) {
  typedef double R2 __attribute__((ext_vector_type(2)));
  constexpr int SL = wide_slots(MB);
  constexpr int LPT = SL <= 8 ? 1 : SL / 8;  // lines of a term, or
  constexpr int TPL = SL <= 8 ? 8 / SL : 1;  // terms of a line
  const int lines = wide_lines(MB, n_a);
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int q = lane >> 3;
  const uint32_t cx0 = (uint32_t)((lane & 7) ^ (q >> 1)) << 4;
  const uint32_t cx1 = (uint32_t)((lane & 7) ^ (4 | (q >> 1))) << 4;
  uint32_t off[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) off[t] = (uint32_t)__shfl((int)boff, 8 * t + q) + ((t & 1) ? cx1 : cx0);
  const uint32_t rbase = (uint32_t)lane * 128u + ((uint32_t)((lane >> 1) & 7) << 4);
  auto issue = [&](int l, int tap) {
    const RIFT_GLOBAL char* ser = uniform_ptr(tab + ((uint64_t)tap * lines + l) * 128u);
    RIFT_LDS unsigned char* dst = stage + (tap & 1) * STAGE_UNIT;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      __builtin_amdgcn_global_load_lds((const RIFT_GLOBAL void*)(ser + off[t]), (RIFT_LDS void*)(dst + t * 1024), 16, 0,
                                       0);
  };
  double data = 0.0;
  issue(0, 0);
#pragma unroll 1
  for (int l0 = 0; l0 < lines; l0 += LPT) {
    double zr[TPL], zi[TPL];
#pragma unroll
    for (int a = 0; a < TPL; ++a) zr[a] = zi[a] = 0.0;
#pragma unroll
    for (int h = 0; h < LPT; ++h) {
      const int l = l0 + h;
      double qx[8], qy[8];
#pragma unroll
      for (int tap = 0; tap < 4; ++tap) {
        // the other buffer's reads have completed: refill it, then wait for this one
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (tap < 3 || l + 1 < lines) {
          issue(tap < 3 ? l : l + 1, (tap + 1) & 3);
          asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        } else {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        const RIFT_LDS unsigned char* src = stage + (tap & 1) * STAGE_UNIT;
        R2 v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = *(const RIFT_LDS R2*)(src + (rbase ^ ((uint32_t)c << 4)));
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          qx[c] = tap == 0 ? wr[0] * v[c].x : fma(wr[tap], v[c].x, qx[c]);
          qy[c] = tap == 0 ? wr[0] * v[c].y : fma(wr[tap], v[c].y, qy[c]);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          pin(qx[c]);
          pin(qy[c]);
        }
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int a = SL <= 8 ? c / SL : 0, m = SL <= 8 ? c % SL : 8 * h + c;
        if (m < 4 * MB) {
          zr[a] = fma(yr[m], qx[c], fma(yi[m], qy[c], zr[a]));
          zi[a] = fma(yr[m], qy[c], fma(-yi[m], qx[c], zi[a]));
        }
      }
    }
#pragma unroll
    for (int a = 0; a < TPL; ++a) {
      const int ta = l0 / LPT * TPL + a;
      if (ta < n_a) {
        const double cx = C[ta * 64 + lane].x, cy = C[ta * 64 + lane].y;
        data = fma(cx, zr[a], fma(cy, zi[a], data));
      }
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  return data;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The sidereal harmonics of the antenna factor times the post-phases,
// C~_n = A_n e^{i n theta}, n = -2..2, theta = g(t_ref) + Omega (t_k - t_ref).
// With e = X + i Y = -e^{-i psi} (e_ra - i e_dec), F(g) = D : e e is
// e^{-2 i psi} times, in E = e^{i g}, p = 1 - sin dec and m = 1 + sin dec,
//   E^2:  p^2 / 4 [(D11 - D00) - 2 i D01]     E^-2: m^2 / 4 [(D11 - D00) + 2 i D01]
//   E:    -cos dec p [D02 + i D12]            E^-1: cos dec m [D02 - i D12]
//   1:    p m [(D00 + D11) / 2 - D22]
// (p m = cos^2 dec): about 60 operations a detector, where the five-point
// transform of F at five hour angles takes 500.
__device__ __forceinline__ void rotation_terms(const double* dten, double sd, double cd, double s2p, double c2p,
                                               double ec, double es, double* cr, double* ci) {
  const double p = 1.0 - sd, m = 1.0 + sd;
  const double dd = dten[1] - dten[0];
  const double e2c = ec * ec - es * es, e2s = 2.0 * ec * es;
  // e^{-2 i psi} e^{i n theta}
  const double fr[5] = {c2p * e2c - s2p * e2s, c2p * ec - s2p * es, c2p, c2p * ec + s2p * es, c2p * e2c + s2p * e2s};
  const double fi[5] = {-c2p * e2s - s2p * e2c, -c2p * es - s2p * ec, -s2p, c2p * es - s2p * ec,
                        c2p * e2s - s2p * e2c};
  const double w2 = 0.25 * p * p, w1 = -0.5 * cd * p, w0 = p * m, v1 = 0.5 * cd * m, v2 = 0.25 * m * m;
  const double ar[5] = {v2 * dd, v1 * dten[4], w0 * (0.5 * (dten[0] + dten[1]) - dten[2]), w1 * dten[4], w2 * dd};
  const double ai[5] = {v2 * dten[3], -v1 * dten[5], 0.0, w1 * dten[5], -w2 * dten[3]};
#pragma unroll
  for (int n = 0; n < 5; ++n) {
    cr[n] = ar[n] * fr[n] - ai[n] * fi[n];
    ci[n] = ar[n] * fi[n] + ai[n] * fr[n];
  }
}

// The pair forms of two terms a <= b, G_ab = Y^H U_ab Y and H_ab = Y^T V_ab Y, in
// the harmonic basis of class L: each of Re G, Im G, Re H, Im H is a trigonometric
// polynomial in (incl, phi) of degree 2L in each, with the parity that d_i d_j
// has in incl, so it lies in the static path's real basis (145 functions at L = 4:
// 580 coefficients a pair, where 21 modes have 1764 entries).  Summed per harmonic
// q in phi: the rows of one q are consecutive and q increases
// along them (basis_row), so
// g[c] += cos(q phi) sum_n C[(n, cos)][c] T_n(incl)
//       + sin(q phi) sum_n C[(n, sin)][c] T_n(incl),
// T_n = cos(n incl) for even q and sin(n incl) for odd q (q = 0: the first
// sum alone), with e^{i q phi} advanced by one factor e^{i phi} per q.
// Every row's kind and degrees are template constants; no product of basis
// values is formed, so only the cos(n incl), sin(n incl) tables stay live
// across the pairs.
template <int L>
struct HarmForms {
  static constexpr int B = Cls<L>::B;
  static constexpr int NC = 4 * B;              // coefficients of one block
  static constexpr int CH = 16;                 // one 128-byte chunk: four rows
  static constexpr int NCH = (NC + CH - 1) / CH;
  struct Run {
    double pc[4], ps[4];  // the two sums of the current q
    double er, ei;        // e^{i q phi}
  };
  template <int J>
  static __device__ __forceinline__ void term(const double* e, const double* cn, const double* sn, double cf,
                                              double sf, double* g, Run& R) {
    if constexpr (J < B) {
      constexpr int rb = basis_row<L>(J);
      constexpr int kind = rb & 15, nn = (rb >> 4) & 255, q = rb >> 12;
      constexpr bool last = (J + 1 == B) || ((basis_row<L>(J + 1) >> 12) != q);
      const double tn = (kind == 3 || kind == 4) ? sn[nn] : cn[nn];
      if constexpr (kind == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k] = fma(e[k], tn, g[k]);
      } else {
        double* acc = (kind == 1 || kind == 3) ? R.pc : R.ps;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = fma(e[k], tn, acc[k]);
        if constexpr (last) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            g[k] = fma(R.pc[k], R.er, fma(R.ps[k], R.ei, g[k]));
            R.pc[k] = 0.0;
            R.ps[k] = 0.0;
          }
          const double nr = R.er * cf - R.ei * sf, ni = R.er * sf + R.ei * cf;
          R.er = nr;
          R.ei = ni;
        }
      }
    }
  }
  // The uniform coefficients stream through SGPRs in 128-byte chunks, each
  // chunk prefetched while the previous one is used (the static path's
  // scheme): the wait for a chunk comes before the next chunk is issued, and
  // the accumulators are pinned after each chunk's FMAs so that those FMAs
  // stay ahead of the next wait.
  template <int C>
  static __device__ __forceinline__ void ld(double (&buf)[CH], const RIFT_CONST double* c) {
    const RIFT_CONST double* p = c + C * CH;
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (C * CH + i < NC) buf[i] = p[i];
  }
  template <int C>
  static __device__ __forceinline__ void wait(const double (&buf)[CH]) {
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (C * CH + i < NC) pin_s(buf[i]);
  }
  template <int C>
  static __device__ __forceinline__ void step(const RIFT_CONST double* c, double (&cur)[CH], double (&nxt)[CH],
                                              const double* cn, const double* sn, double cf, double sf, double* g,
                                              Run& R) {
    if constexpr (C < NCH) {
      wait<C>(cur);
      if constexpr (C + 1 < NCH) ld<C + 1>(nxt, c);
      term<4 * C>(cur, cn, sn, cf, sf, g, R);
      term<4 * C + 1>(cur + 4, cn, sn, cf, sf, g, R);
      term<4 * C + 2>(cur + 8, cn, sn, cf, sf, g, R);
      term<4 * C + 3>(cur + 12, cn, sn, cf, sf, g, R);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pin(g[k]);
        pin(R.pc[k]);
        pin(R.ps[k]);
      }
      step<C + 1>(c, nxt, cur, cn, sn, cf, sf, g, R);
    }
  }
  static __device__ __forceinline__ void run(const RIFT_CONST double* c, const double* cn, const double* sn,
                                             double cf, double sf, double* g) {
    Run R;
#pragma unroll
    for (int k = 0; k < 4; ++k) R.pc[k] = R.ps[k] = 0.0;
    R.er = cf;  // the first group after q = 0 is q = 1
    R.ei = sf;
    double bA[CH], bB[CH];
    ld<0>(bA, c);
    step<0>(c, bA, bB, cn, sn, cf, sf, g, R);
  }
};

// Harmonic-basis coefficients of the pair forms, one block per (detector,
// pair a <= b): Re G, Im G, Re H, Im H of the block sampled on an NG x NG
// grid of (incl, phi) over [0, 2 pi)^2, NG = 4L + 4 (more than twice the
// degree 2L in each), then projected on the basis rows (discrete
// orthogonality on that grid).  Every angle on the grid is a multiple of
// 2 pi / NG, so cos and sin come from one table of NG entries each; the
// block's U and V entries are staged in LDS; a thread per grid point, then
// each basis row's projection split over WIDE_BASIS_BLOCK / B threads.  U, V in the caller's order
// [K][A][A] complex; out [K][pair][B][4].
template <int L>
__global__ void k_wide_basis(WideDesc D, const double* __restrict__ U, const double* __restrict__ V,
                             double* __restrict__ out) {
  constexpr int NG = 4 * L + 4, B = Cls<L>::B, MX = Cls<L>::MAXM;
  constexpr int PS = WIDE_BASIS_BLOCK / B;  // threads per basis row in the projection
  __shared__ double g[4][NG * NG];
  __shared__ double part[PS][B][4];
  __shared__ double ct[NG], st[NG];
  __shared__ double uv[MX * MX][4];
  const int k = blockIdx.x / D.npairs, pr = blockIdx.x - k * D.npairs;
  int a = 0, rem = pr;
  while (rem >= D.n_a - a) {
    rem -= D.n_a - a;
    ++a;
  }
  const int b = a + rem;
  const int M = D.M, A = D.n_a * D.M;
  for (int j = threadIdx.x; j < NG; j += blockDim.x) {
    double sj, cj;
    sincospi(2.0 * j / NG, &sj, &cj);
    ct[j] = cj;
    st[j] = sj;
  }
  for (int e = threadIdx.x; e < M * M; e += blockDim.x) {
    const int i = e / M, j = e - (e / M) * M;
    const int64_t o = 2 * (((int64_t)k * A + a * M + D.perm[i]) * A + b * M + D.perm[j]);
    uv[e][0] = U[o];
    uv[e][1] = U[o + 1];
    uv[e][2] = V[o];
    uv[e][3] = V[o + 1];
  }
  __syncthreads();
  // index of the angle n * (2 pi c / NG) in the tables
  auto ix = [](int n, int c) { return ((n * c) % NG + NG) % NG; };
  for (int gp = threadIdx.x; gp < NG * NG; gp += blockDim.x) {
    const int pi_ = gp / NG, pf = gp - (gp / NG) * NG;
    double yr[MX], yi[MX];
#pragma unroll
    for (int i = 0; i < MX; ++i) {
      yr[i] = yi[i] = 0.0;
      if (i < M) {
        double d = 0.0;
        for (int q = 0; q <= L; ++q) d += D.ycoef[i][q] * (D.odd[i] ? st[ix(q, pi_)] : ct[ix(q, pi_)]);
        const int r = ix(D.m[i], pf);
        yr[i] = d * ct[r];
        yi[i] = d * st[r];
      }
    }
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < MX; ++i) {
      if (i < M) {
        double tr = 0.0, ti = 0.0, wr = 0.0, wi = 0.0;
#pragma unroll
        for (int j = 0; j < MX; ++j) {
          if (j < M) {
            const double* e = uv[i * M + j];
            tr += e[0] * yr[j] - e[1] * yi[j];
            ti += e[0] * yi[j] + e[1] * yr[j];
            wr += e[2] * yr[j] - e[3] * yi[j];
            wi += e[2] * yi[j] + e[3] * yr[j];
          }
        }
        v[0] += yr[i] * tr + yi[i] * ti;
        v[1] += yr[i] * ti - yi[i] * tr;
        v[2] += yr[i] * wr - yi[i] * wi;
        v[3] += yr[i] * wi + yi[i] * wr;
      }
    }
    for (int c = 0; c < 4; ++c) g[c][gp] = v[c];
  }
  __syncthreads();
  // each row's sum over the grid split over PS threads, then reduced
  for (int w = threadIdx.x; w < PS * B; w += blockDim.x) {
    const int r = w % B, sp = w / B;
    const int rb = basis_row<L>(r);
    const int kind = rb & 15, nn = (rb >> 4) & 255, q = rb >> 12;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int gp = sp; gp < NG * NG; gp += PS) {
      const int pi_ = gp / NG, pf = gp - (gp / NG) * NG;
      const double ti = (kind >= 3) ? st[ix(nn, pi_)] : ct[ix(nn, pi_)];
      const double tf = (kind == 0) ? 1.0 : (kind == 1 || kind == 3) ? ct[ix(q, pf)] : st[ix(q, pf)];
      const double t = ti * tf;
      for (int c = 0; c < 4; ++c) acc[c] += g[c][gp] * t;
    }
    for (int c = 0; c < 4; ++c) part[sp][r][c] = acc[c];
  }
  __syncthreads();
  for (int r = threadIdx.x; r < B; r += blockDim.x) {
    const int rb = basis_row<L>(r);
    const int nn = (rb >> 4) & 255, q = rb >> 12;
    const double norm = 1.0 / ((double)NG * NG * (nn == 0 ? 1.0 : 0.5) * (q == 0 ? 1.0 : 0.5));
    double* o = out + ((int64_t)blockIdx.x * B + r) * 4;
    for (int c = 0; c < 4; ++c) {
      double v = 0.0;
      for (int sp = 0; sp < PS; ++sp) v += part[sp][r][c];
      o[c] = v * norm;
    }
  }
}

// sin and cos of |x| <= 1 by their Taylor series through x^19 / 19! and
// x^18 / 18! (truncation below 1e-17): the rotation over the light-travel
// time, Omega (t_k - t_ref), which the validation keeps within one radian.
__device__ __forceinline__ void sincos_small(double x, double* s, double* c) {
  const double x2 = x * x;
  double ps = -1.0 / 121645100408832000.0;  // -1/19!
  ps = fma(ps, x2, 1.0 / 355687428096000.0);
  ps = fma(ps, x2, -1.0 / 1307674368000.0);
  ps = fma(ps, x2, 1.0 / 6227020800.0);
  ps = fma(ps, x2, -1.0 / 39916800.0);
  ps = fma(ps, x2, 1.0 / 362880.0);
  ps = fma(ps, x2, -1.0 / 5040.0);
  ps = fma(ps, x2, 1.0 / 120.0);
  ps = fma(ps, x2, -1.0 / 6.0);
  *s = fma(ps * x2, x, x);
  double pc = 1.0 / 6402373705728000.0;  // 1/18!
  pc = fma(pc, x2, -1.0 / 20922789888000.0);
  pc = fma(pc, x2, 1.0 / 87178291200.0);
  pc = fma(pc, x2, -1.0 / 479001600.0);
  pc = fma(pc, x2, 1.0 / 3628800.0);
  pc = fma(pc, x2, -1.0 / 40320.0);
  pc = fma(pc, x2, 1.0 / 720.0);
  pc = fma(pc, x2, -1.0 / 24.0);
  pc = fma(pc, x2, 0.5);
  *c = fma(-pc, x2, 1.0);
}

// The complete set of l <= 4 (21 modes) has a second form of the quadratic term:
// the harmonic forms of the pairs on the vector unit, 52 kflop a sample at five
// terms where the real form's tiles take 132.  It is bound by the latency of its
// scalar stream, the same from one wavefront to two per SIMD, where the real form
// takes the matrix cores' time twice: it takes calls that put two wavefronts on a
// SIMD, of eight terms and more, and of five and more while they are one or two
// rounds of the chip.  Measured (3 detectors, us; real form, harmonic form): 12
// terms, 65536 samples 1571, 2213; 131072 3078, 2388; 200k 5673, 4495; 300k 6969,
// 6772.  21 terms, 20k 4353, 6064; 65536 8169, 6100; 100k 9488, 6230.  Eight, 100k
// 1445, 1162; 300k 3354, 3417.  Five, 131072 697, 641; 300k 1496, 1662.  With 17
// modes the two meet (12 terms, 131072: 2246, 2255).
constexpr int WIDE_HARMONIC_M = 21;
bool wide_harmonic(int M, int lmax, int n_a, int64_t n) {
  if (M != WIDE_HARMONIC_M || lmax > 4) return false;
  if (n_a > 12) return n > 49152;
  return n > 65536 && (n_a >= 8 || (n_a >= 5 && n <= 262144));
}

// Dynamic LDS of a wavefront: the staging of the data term's rows (the
// harmonics' exchange reuses it), then the coefficients.
__host__ __device__ constexpr int wide_stage_bytes(bool packed, int HL) { return packed ? STAGE_WAVE : (HL ? 0 : 4 * 64 * 16); }

// One wavefront per block: its LDS (21 KB at five terms) then packs seven to a
// CU, within the registers of two per SIMD.
template <int MB, bool PACKED, int HL = 0>
__global__ void __launch_bounds__(64, 2) k_wide(WideDesc D, const double* __restrict__ theta, int64_t n,
                                                const double* __restrict__ lnw, double* __restrict__ lnL,
                                                double* __restrict__ part) {
  typedef double D4 __attribute__((ext_vector_type(4)));
  constexpr int MC = 4 * MB;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ MS sh[1];
  RIFT_LDS unsigned char* stage = (RIFT_LDS unsigned char*)smem;
  const WideCoef C = (WideCoef)(stage + wide_stage_bytes(PACKED, HL));
  const int t = threadIdx.x, col = t & 15, quad = t >> 4;
  const int64_t i0 = (int64_t)blockIdx.x * 64 + t;
  const bool live = i0 < n;
  const int64_t i = live ? i0 : n - 1;
  const RIFT_GLOBAL double* th = as_global(theta) + i;
  const double ra = th[0], dec = th[n], psi = th[2 * n], incl = th[3 * n], phi = th[4 * n];
  const double tref = th[5 * n], dist = th[6 * n];
  const int K = D.K, M = D.M, n_t = D.n_t, n_a = D.n_a;
  const bool rot = D.response == RIFT_RESP_ROTATION || D.response == RIFT_RESP_ROTATION_DELAY;
  const bool drift = D.response == RIFT_RESP_ROTATION_DELAY && n_a > 5;

  // sky frame at t_ref (the rotation response advances the sidereal angle)
  const double gm = rot ? D.gmst + D.omega * tref : D.gmst;
  const double gref = gm - ra;
  const double a5[5] = {gref, dec, psi, incl, phi};
  double s5[5], c5[5];
  sincos_many<5>(a5, s5, c5);
  const double sg = s5[0], cg = c5[0], sd = s5[1], cd = c5[1], sp = s5[2], cp = c5[2];
  double X[3], Y3[3], N[3];
  axes(sg, cg, sd, cd, sp, cp, X, Y3, N);

  // harmonics Y_i = d_i(incl) e^{i m_i phi}, internal (m-sorted) modes
  double yr[MC], yi[MC];
  {
    const double si = s5[3], ci = c5[3], sf = s5[4], cf = c5[4];
    double cn[LMAXC + 1], sn[LMAXC + 1];
    double c0 = 1.0, c1 = ci, s0 = 0.0, s1 = si;
#pragma unroll
    for (int q = 0; q <= LMAXC; ++q) {
      cn[q] = (q == 0) ? c0 : c1;
      sn[q] = (q == 0) ? s0 : s1;
      if (q > 0) {
        const double c2 = 2.0 * ci * c1 - c0, s2 = 2.0 * ci * s1 - s0;
        c0 = c1;
        c1 = c2;
        s0 = s1;
        s1 = s2;
      }
    }
    C2<double> ph;
    ph.x = 1.0;
    ph.y = 0.0;
    const int mmin = D.m[0];
    for (int q = 0; q < -mmin; ++q) phase_down(ph, cf, sf);
    int mc = mmin < 0 ? mmin : 0;
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      yr[j] = yi[j] = 0.0;
      if (j < M) {
        const int mj = D.m[j];
        while (mc < mj) {
          phase_up(ph, cf, sf);
          ++mc;
        }
        double d = 0.0;
        if (D.odd[j]) {
#pragma unroll
          for (int q = 1; q <= LMAXC; ++q) d += D.ycoef[j][q] * sn[q];
        } else {
#pragma unroll
          for (int q = 0; q <= LMAXC; ++q) d += D.ycoef[j][q] * cn[q];
        }
        yr[j] = d * ph.x;
        yi[j] = d * ph.y;
      }
    }
  }
  // detector k's arrival time, its coefficients into this lane's column
  auto coefficients = [&](int k) {
    const double tk = tref - (D.rpos[k][0] * N[0] + D.rpos[k][1] * N[1] + D.rpos[k][2] * N[2]);
    auto set = [&](int a, double re, double im) {
      C[a * 64 + t].x = re;
      C[a * 64 + t].y = im;
    };
    if (rot) {
      // e^{i theta_k} = e^{i g(t_ref)} e^{i Omega (t_k - t_ref)}
      double sdl, cdl;
      sincos_small(D.omega * (tk - tref), &sdl, &cdl);
      double c0r[5], c0i[5];
      rotation_terms(D.dten[k], sd, cd, 2.0 * sp * cp, cp * cp - sp * sp, cg * cdl - sg * sdl, sg * cdl + cg * sdl, c0r,
                     c0i);
#pragma unroll
      for (int a = 0; a < 5; ++a) set(a, c0r[a], c0i[a]);
      if (drift) {
        // first order in the delay drift (Path B, p = 1).  The drift's
        // harmonics in the modulation phase, -dt: m = -1, 0, +1 from
        // rho e^{i g(t_ref)}, rho = r_x + i r_y.  With the post-phases
        // folded in, C~_(1, n) = sum_m C~_(0, n - m) D_m e^{i m Omega (t_k - t_ref)}
        // for n = -3 .. 3
        const double rer = D.rpos[k][0] * cg - D.rpos[k][1] * sg, rei = D.rpos[k][0] * sg + D.rpos[k][1] * cg;
        // D_m e^{i m Omega (t_k - t_ref)}, m = -1, 0, +1
        const double hr = 0.5 * cd * rer, hi = 0.5 * cd * rei;
        const double dmr[3] = {hr * cdl - hi * sdl, -cd * rer, hr * cdl - hi * sdl};
        const double dmi[3] = {hr * (-sdl) - hi * cdl, 0.0, hr * sdl + hi * cdl};
#pragma unroll
        for (int b = 0; b < 7; ++b) {
          double cr = 0.0, ci = 0.0;
#pragma unroll
          for (int m = -1; m <= 1; ++m) {
            const int q = b - 3 - m;
            if (q < -2 || q > 2) continue;
            cr += c0r[q + 2] * dmr[m + 1] - c0i[q + 2] * dmi[m + 1];
            ci += c0r[q + 2] * dmi[m + 1] + c0i[q + 2] * dmr[m + 1];
          }
          set(5 + b, cr, ci);
        }
        if (n_a >= 21) {
          // order 2: the drift's square, (D~ * D~)_m for m = -2..2, and
          // C~_(2, n) = 1/2 sum_m C~_(0, n - m) (D~ * D~)_m for n = -4..4
          double d2r[5], d2i[5];
#pragma unroll
          for (int m = 0; m < 5; ++m) d2r[m] = d2i[m] = 0.0;
#pragma unroll
          for (int m1 = 0; m1 < 3; ++m1)
#pragma unroll
            for (int m2 = 0; m2 < 3; ++m2) {
              d2r[m1 + m2] += dmr[m1] * dmr[m2] - dmi[m1] * dmi[m2];
              d2i[m1 + m2] += dmr[m1] * dmi[m2] + dmi[m1] * dmr[m2];
            }
#pragma unroll
          for (int b = 0; b < 9; ++b) {
            double cr = 0.0, ci = 0.0;
#pragma unroll
            for (int m = -2; m <= 2; ++m) {
              const int q = b - 4 - m;
              if (q < -2 || q > 2) continue;
              cr += c0r[q + 2] * d2r[m + 2] - c0i[q + 2] * d2i[m + 2];
              ci += c0r[q + 2] * d2i[m + 2] + c0i[q + 2] * d2r[m + 2];
            }
            set(12 + b, 0.5 * cr, 0.5 * ci);
          }
        }
      }
    } else {
      const double* ax = D.arms[k][0];
      const double* ay = D.arms[k][1];
      const double xX = X[0] * ax[0] + X[1] * ax[1] + X[2] * ax[2];
      const double xY = Y3[0] * ax[0] + Y3[1] * ax[1] + Y3[2] * ax[2];
      const double yX = X[0] * ay[0] + X[1] * ay[1] + X[2] * ay[2];
      const double yY = Y3[0] * ay[0] + Y3[1] * ay[1] + Y3[2] * ay[2];
      const double exr = xX * xX - xY * xY, exi = 2.0 * xX * xY;
      const double eyr = yX * yX - yY * yY, eyi = 2.0 * yX * yY;
      const double ux = N[0] * ax[0] + N[1] * ax[1] + N[2] * ax[2];
      const double uy = N[0] * ay[0] + N[1] * ay[1] + N[2] * ay[2];
      double px = 1.0, py = 1.0;
      for (int a = 0; a < n_a; ++a) {
        set(a, 0.5 * (px * exr - py * eyr), 0.5 * (px * exi - py * eyi));
        px *= ux;
        py *= uy;
      }
    }
    return tk;
  };

  double data = 0.0, quadratic = 0.0;
  bool bad = false;
#pragma unroll 1
  for (int k = 0; k < K; ++k) {
    const double tk = coefficients(k);
    // four-point Lagrange stencil at t_k (taps outside the window read zero)
    double u = (tk - D.t0) * D.inv_dt;
    if (!(fabs(u) <= 1.0e300)) {
      bad = true;
      u = 0.0;
    }
    u = fmin(fmax(u, -8.0), (double)n_t + 8.0);
    const double jf = floor(u);
    const double s = u - jf;
    const int j0 = (int)jf - 1;
    double w[4];
    lagrange4(s, w);
#pragma unroll
    for (int tap = 0; tap < 4; ++tap)
      if (j0 + tap < 0 || j0 + tap >= n_t) w[tap] = 0.0;
    // the four rows read are jc .. jc+3, inside the window; row jc + r carries
    // tap r + jc - j0 (weight 0 when that is not a tap or lies outside)
    const int jc = j0 < 0 ? 0 : (j0 > n_t - 4 ? n_t - 4 : j0);
    double wr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tp = r + jc - j0;
      double v = 0.0;
#pragma unroll
      for (int tap = 0; tap < 4; ++tap) v = (tp == tap) ? w[tap] : v;
      wr[r] = v;
    }
    // data term: Re sum_a conj(C~_a) sum_i conj(Y_i) Qhat_{a,i}
    if constexpr (PACKED) {
      const int lines = wide_lines(MB, n_a);
      const RIFT_GLOBAL char* tab = (const RIFT_GLOBAL char*)as_global(D.Qrows) + (uint64_t)k * n_t * lines * 128u;
      data += wide_data<MB>(tab, (uint32_t)jc * (uint32_t)(lines * 128), n_a, stage, wr, yr, yi, C);
    } else {
      for (int a = 0; a < n_a; ++a) {
        double zr = 0.0, zi = 0.0;
#pragma unroll
        for (int j = 0; j < MC; ++j) {
          if (j < M) {
            const RIFT_GLOBAL double* q =
                as_global(D.Q) + 2 * ((((int64_t)k * n_a + a) * M + D.perm[j]) * (int64_t)n_t + jc);
            double qr = 0.0, qi = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              qr += wr[r] * q[2 * r];
              qi += wr[r] * q[2 * r + 1];
            }
            // conj(Y) Qhat
            zr += yr[j] * qr + yi[j] * qi;
            zi += yr[j] * qi - yi[j] * qr;
          }
        }
        // Re[conj(C~_a) z]
        data += C[a * 64 + t].x * zr + C[a * 64 + t].y * zi;
      }
    }
    if constexpr (HL > 0) {
      // model-norm term over pairs a <= b.  The angles' values are rebuilt per
      // detector, the phase sequence per pair: hoisted, they would hold their
      // registers through the reads
      double co = c5[3], so = s5[3];
      pin(co);
      pin(so);
      double cn[2 * HL + 1], sn[2 * HL + 1];
      cn[0] = 1.0;
      sn[0] = 0.0;
      cn[1] = co;
      sn[1] = so;
#pragma unroll
      for (int q = 2; q <= 2 * HL; ++q) {
        cn[q] = 2.0 * co * cn[q - 1] - cn[q - 2];
        sn[q] = 2.0 * co * sn[q - 1] - sn[q - 2];
      }
      constexpr int BS = 4 * Cls<(HL > 0 ? HL : 2)>::B;
      const RIFT_CONST double* blk = as_const(D.S) + (int64_t)k * D.npairs * BS;
#pragma unroll 1
      for (int a = 0; a < n_a; ++a) {
#pragma unroll 1
        for (int b = a; b < n_a; ++b, blk += BS) {
          double g[4] = {0.0, 0.0, 0.0, 0.0};  // Re G, Im G, Re H, Im H
          double cf = c5[4], sf = s5[4];
          pin(cf);
          pin(sf);
          HarmForms<(HL > 0 ? HL : 2)>::run(opaque(blk), cn, sn, cf, sf, g);
          const double ar = C[a * 64 + t].x, ai = C[a * 64 + t].y, br = C[b * 64 + t].x, bi = C[b * 64 + t].y;
          // conj(C_a) C_b G_ab and C_a C_b H_ab, counted twice off the diagonal
          const double pr = ar * br + ai * bi, pim = ar * bi - ai * br;
          const double qr = ar * br - ai * bi, qim = ar * bi + ai * br;
          quadratic += (a == b ? 1.0 : 2.0) * ((pr * g[0] - pim * g[1]) + (qr * g[2] - qim * g[3]));
        }
      }
    }
  }

  if constexpr (HL == 0) {
    // the harmonics as the matrix tiles take them: sample 16 s + col, mode 4 mb + quad
    double vr[4][MB], vi[4][MB];
    {
      RIFT_LDS double2* ex = (RIFT_LDS double2*)stage;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        wave_sync();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          ex[q * 64 + t].x = yr[4 * mb + q];
          ex[q * 64 + t].y = yi[4 * mb + q];
        }
        wave_sync();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          vr[s][mb] = ex[quad * 64 + 16 * s + col].x;
          vi[s][mb] = ex[quad * 64 + 16 * s + col].y;
        }
      }
    }
    // model-norm term: per detector sum_t c_t^T (S c)_t, this lane's share of it
    // the components (step, quad) of samples 16 s + col
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int steps = wide_steps(MB, n_a), tiles = wide_tiles(MB, n_a);
    typedef double R2 __attribute__((ext_vector_type(2)));
    const RIFT_GLOBAL R2* A = (const RIFT_GLOBAL R2*)as_global(D.S) + t;
    R2 nxt = A[0];
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      if (K > 1) {
        wave_sync();
        (void)coefficients(k);
      }
      wave_sync();
#pragma unroll 1
      for (int tl = 0; tl < tiles; ++tl) {
        D4 d[4];
        double keep[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          d[s] = D4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int r = 0; r < 4; ++r) keep[s][r] = 0.0;
        }
        const int b0 = 4 * tl;
        int a = b0 / (2 * MB);
#pragma unroll 1
        for (int b = a * 2 * MB; b < steps; ++a) {
          double cr[4], ci[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            cr[s] = C[a * 64 + 16 * s + col].x;
            ci[s] = C[a * 64 + 16 * s + col].y;
          }
#pragma unroll
          for (int mb = 0; mb < MB; ++mb, b += 2) {
            if (b < b0) continue;
            const R2 cur = nxt;
            A += 64;
            nxt = A[0];  // one pair past the end is padding
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              const double xr = cr[s] * vr[s][mb] - ci[s] * vi[s][mb], xi = cr[s] * vi[s][mb] + ci[s] * vr[s][mb];
              d[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur.x, xr, d[s], 0, 0, 0);
              d[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur.y, xi, d[s], 0, 0, 0);
              if (b == b0) {
                keep[s][0] = xr;
                keep[s][1] = xi;
              } else if (b == b0 + 2) {
                keep[s][2] = xr;
                keep[s][3] = xi;
              }
            }
          }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[s] = fma(d[s][r], keep[s][r], acc[s]);
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      acc[s] += __shfl_xor(acc[s], 16);
      acc[s] += __shfl_xor(acc[s], 32);
    }
    // sample t = 16 quad + col
    quadratic = quad == 0 ? acc[0] : (quad == 1 ? acc[1] : (quad == 2 ? acc[2] : acc[3]));
  }
  const double x = D.d_ref / dist;
  double l = x * data - 0.25 * x * x * quadratic;
  if (bad) l = __builtin_nan("");
  if (live && lnL) as_global_w(lnL)[i] = l;
  if (part) {
    MS m;
    m.m = -__builtin_inf();
    m.s = 0.0;
    if (live) m = ms_push(m, l + (lnw ? as_global(lnw)[i] : 0.0));
    const MS r = ms_block(m, sh);
    if (t == 0) {
      part[2 * (int64_t)blockIdx.x] = r.m;
      part[2 * (int64_t)blockIdx.x + 1] = r.s;
    }
  }
}

template <int MB>
void launch_wide(const WideDesc& D, bool packed, bool harmonic, const double* U, const double* V, double* form,
                 double* rows, const double* theta, int64_t n, const double* lnw, double* lnL, double* part,
                 hipStream_t st) {
  constexpr int HL = MB == (WIDE_HARMONIC_M + 3) / 4 ? 4 : 0;
  if (harmonic) {
    hipLaunchKernelGGL(k_wide_basis<4>, dim3((unsigned)(D.K * D.npairs)), dim3(WIDE_BASIS_BLOCK), 0, st, D, U, V, form);
  } else {
    const int64_t total = (int64_t)D.K * wide_pairs(wide_steps(MB, D.n_a), wide_tiles(MB, D.n_a)) * 128;
    hipLaunchKernelGGL(k_wide_form<MB>, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 4096)), dim3(256), 0, st,
                       D, U, V, form);
  }
  const dim3 grid((unsigned)((n + 63) / 64)), block(64);
  const size_t lds = wide_stage_bytes(packed, harmonic ? HL : 0) + (size_t)D.n_a * 64 * 16;
  if (packed) {
    const int lines = wide_lines(MB, D.n_a);
    hipLaunchKernelGGL(k_wide_rows, dim3((unsigned)((D.n_t + WIDE_QT - 1) / WIDE_QT), (unsigned)D.K,
                                         (unsigned)std::min(lines, 4)),
                       dim3(256), 0, st, D, wide_slots(MB), lines, rows);
    hipLaunchKernelGGL((k_wide<MB, true>), grid, block, lds, st, D, theta, n, lnw, lnL, part);
  } else if (harmonic) {
    hipLaunchKernelGGL((k_wide<MB, false, HL>), grid, block, lds, st, D, theta, n, lnw, lnL, part);
  } else {
    hipLaunchKernelGGL((k_wide<MB, false>), grid, block, lds, st, D, theta, n, lnw, lnL, part);
  }
}

// ln Z and n_eff from the blocks' (max, sum) pairs, one block, fixed order.
__global__ void k_wide_merge(double lnN, const double* __restrict__ part, int nb, double* __restrict__ lnZ,
                             double* __restrict__ neff) {
  // the blocks' maximum first, then sums whose exponentials are independent
  __shared__ double sm[WIDE_MERGE / 64];
  double m = -__builtin_inf();
  for (int b = threadIdx.x; b < nb; b += blockDim.x) m = fmax(m, part[2 * b]);
  m = dmax_wave(m);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
  __syncthreads();
  m = sm[0];
  for (int w = 1; w < WIDE_MERGE / 64; ++w) m = fmax(m, sm[w]);
  __syncthreads();
  double s = 0.0;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    const double o = part[2 * b + 1];
    s += o == 0.0 ? 0.0 : o * exp(part[2 * b] - m);  // a NaN sum stays NaN
  }
  s = dsum_wave(s);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = s;
  __syncthreads();
  MS r;
  r.m = m;
  r.s = sm[0];
  for (int w = 1; w < WIDE_MERGE / 64; ++w) r.s += sm[w];
  if (threadIdx.x == 0) {
    double z;
    if (r.s != r.s) z = __builtin_nan("");
    else if (r.m == -__builtin_inf()) z = -__builtin_inf();
    else z = r.m + log(r.s) - lnN;
    lnZ[0] = z;
    if (neff) neff[0] = (r.m == -__builtin_inf() && r.s == r.s) ? 0.0 : r.s;
  }
}

int validate_wide(const rift_ile_point_wide* pt) {
  if (!pt) return RIFT_EINVAL;
  if (pt->n_det < 1 || pt->n_det > RIFT_ILE_MAX_DET) return RIFT_EINVAL;
  if (pt->n_modes < 1 || pt->n_modes > RIFT_ILE_MAX_MODES) return RIFT_EINVAL;
  if (pt->n_t < 4 || pt->n_t > RIFT_ILE_MAX_NT) return RIFT_EINVAL;
  if (pt->response == RIFT_RESP_ROTATION) {
    if (pt->n_terms != 5) return RIFT_EINVAL;
    if (!std::isfinite(pt->omega)) return RIFT_EINVAL;
  } else if (pt->response == RIFT_RESP_ROTATION_DELAY) {
    if (pt->n_terms != 5 && pt->n_terms != 12 && pt->n_terms != 21) return RIFT_EINVAL;
    if (!std::isfinite(pt->omega)) return RIFT_EINVAL;
  } else if (pt->response == RIFT_RESP_ARMS) {
    if (pt->n_terms < 1 || pt->n_terms > WIDE_ARMS_MAX_TERMS || !pt->det_arms) return RIFT_EINVAL;
    for (int a = 0; a < 6 * pt->n_det; ++a)
      if (!std::isfinite(pt->det_arms[a])) return RIFT_EINVAL;
  } else {
    return RIFT_EINVAL;
  }
  if (!pt->lm || !pt->Q || !pt->U || !pt->V || !pt->det_tensor || !pt->det_pos) return RIFT_EINVAL;
  if ((((uintptr_t)pt->Q) | ((uintptr_t)pt->U) | ((uintptr_t)pt->V)) & 7u) return RIFT_EINVAL;
  if (!std::isfinite(pt->t0) || !std::isfinite(pt->dt) || !(pt->dt > 0.0)) return RIFT_EINVAL;
  if (!std::isfinite(pt->gmst_rad) || !std::isfinite(pt->d_ref) || !(pt->d_ref > 0.0)) return RIFT_EINVAL;
  for (int i = 0; i < pt->n_modes; ++i) {
    const int l = pt->lm[2 * i], m = pt->lm[2 * i + 1];
    if (l < 2 || l > RIFT_ILE_MAX_L || m < -l || m > l) return RIFT_EINVAL;
    for (int j = 0; j < i; ++j)
      if (pt->lm[2 * j] == l && pt->lm[2 * j + 1] == m) return RIFT_EINVAL;
  }
  for (int a = 0; a < 9 * pt->n_det; ++a)
    if (!std::isfinite(pt->det_tensor[a])) return RIFT_EINVAL;
  for (int a = 0; a < 3 * pt->n_det; ++a)
    if (!std::isfinite(pt->det_pos[a])) return RIFT_EINVAL;
  // rotation: the turn over the light-travel time, Omega |r_k|, stays within
  // one radian (the post-phase is evaluated by a series on that range)
  if (pt->response == RIFT_RESP_ROTATION || pt->response == RIFT_RESP_ROTATION_DELAY)
    for (int k = 0; k < pt->n_det; ++k) {
      const double* r = pt->det_pos + 3 * k;
      if (!(fabs(pt->omega) * sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]) <= 1.0)) return RIFT_EINVAL;
    }
  return RIFT_OK;
}

// One call: description to the device, the sample kernel, optionally the merge.
int wide_run(const rift_ile_point_wide* pt, int64_t n, const double* theta, const double* lnw, double* lnL,
             double* lnZ, double* neff, void* stream) {
  int rc = validate_wide(pt);
  if (rc) return rc;
  if (n < 0) return RIFT_EINVAL;
  if (n == 0) return lnZ ? RIFT_EINVAL : RIFT_OK;
  auto bad_ptr = [](const void* p) { return !p || (((uintptr_t)p) & 7u); };
  if (bad_ptr(theta) || (lnL && bad_ptr(lnL)) || (lnw && bad_ptr(lnw)) || (lnZ && bad_ptr(lnZ)) ||
      (neff && bad_ptr(neff)))
    return RIFT_EINVAL;
  if (!lnL && !lnZ) return RIFT_EINVAL;
  const int64_t nb = (n + 63) / 64;
  if (nb > 0x7fffffff) return RIFT_EUNSUPPORTED;
  WideDesc D;
  memset(&D, 0, sizeof(D));
  D.K = pt->n_det;
  D.M = pt->n_modes;
  D.n_t = pt->n_t;
  D.n_a = pt->n_terms;
  D.response = pt->response;
  D.t0 = pt->t0;
  D.inv_dt = 1.0 / pt->dt;
  D.gmst = pt->gmst_rad;
  D.omega = (pt->response == RIFT_RESP_ROTATION || pt->response == RIFT_RESP_ROTATION_DELAY) ? pt->omega : 0.0;
  D.d_ref = pt->d_ref;
  for (int k = 0; k < pt->n_det; ++k) {
    const double* d = pt->det_tensor + 9 * k;
    const double six[6] = {d[0], d[4], d[8], d[1] + d[3], d[2] + d[6], d[5] + d[7]};
    for (int a = 0; a < 6; ++a) D.dten[k][a] = six[a];
    for (int a = 0; a < 3; ++a) D.rpos[k][a] = pt->det_pos[3 * k + a];
    if (pt->response == RIFT_RESP_ARMS)
      for (int e = 0; e < 2; ++e)
        for (int a = 0; a < 3; ++a) D.arms[k][e][a] = pt->det_arms[6 * k + 3 * e + a];
  }
  std::vector<int> perm(pt->n_modes);
  for (int i = 0; i < pt->n_modes; ++i) perm[i] = i;
  std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) { return pt->lm[2 * a + 1] < pt->lm[2 * b + 1]; });
  for (int i = 0; i < pt->n_modes; ++i) {
    const int l = pt->lm[2 * perm[i]], m = pt->lm[2 * perm[i] + 1];
    D.perm[i] = perm[i];
    D.m[i] = m;
    D.odd[i] = (m & 1) ? 1 : 0;
    ylm_fourier(l, m, D.ycoef[i]);
  }
  D.Q = pt->Q;
  const int MB = (pt->n_modes + 3) / 4;
  D.npairs = D.n_a * (D.n_a + 1) / 2;
  int lmax = 0;
  for (int i = 0; i < pt->n_modes; ++i) lmax = std::max(lmax, (int)pt->lm[2 * i]);
  const bool harmonic = wide_harmonic(D.M, lmax, D.n_a, n);
  const size_t row_bytes = 128 * (size_t)wide_lines(MB, D.n_a);
  bool packed = !harmonic && wide_packs(D.K, D.M, D.n_a, n) && (uint64_t)D.n_t * row_bytes <= 0xffffffffu;
  // stream-ordered scratch: the repacked rows, the real form's operands (and
  // one pair of steps that is fetched past the end) or the harmonic form's
  // coefficients, the blocks' (max, sum) pairs
  size_t q_bytes = packed ? (size_t)D.K * D.n_t * row_bytes : 0;
  const int steps = wide_steps(MB, D.n_a);
  const size_t form_bytes =
      harmonic ? sizeof(double) * 4 * (size_t)(D.K * D.npairs * Cls<4>::B)
               : sizeof(double) * 128 * (size_t)(D.K * wide_pairs(steps, wide_tiles(MB, D.n_a)) + 1);
  const size_t part_bytes = lnZ ? sizeof(double) * 2 * (size_t)nb : 0;
  hipStream_t st = (hipStream_t)stream;
  char* space = nullptr;
  auto take = [&]() {
    if (hipMallocAsync((void**)&space, q_bytes + form_bytes + part_bytes, st) == hipSuccess) return true;
    (void)hipGetLastError();  // handled here, not by the next launch
    return false;
  };
  bool have = take();
  if (!have && packed) {  // no room for a second copy of the table: its series are read as they are
    packed = false;
    q_bytes = 0;
    have = take();
  }
  if (!have) return RIFT_ENOMEM;
  double* form = (double*)(space + q_bytes);
  double* d_part = lnZ ? (double*)(space + q_bytes + form_bytes) : nullptr;
  D.Qrows = (const double*)space;
  D.S = form;
#define RIFT_WIDE(B) \
  case B: launch_wide<B>(D, packed, harmonic, pt->U, pt->V, form, (double*)space, theta, n, lnw, lnL, d_part, st); break;
  switch (MB) {
    RIFT_WIDE(1)
    RIFT_WIDE(2)
    RIFT_WIDE(3)
    RIFT_WIDE(4)
    RIFT_WIDE(5)
    RIFT_WIDE(6)
    RIFT_WIDE(7)
  }
#undef RIFT_WIDE
  if (lnZ)
    hipLaunchKernelGGL(k_wide_merge, dim3(1), dim3(WIDE_MERGE), 0, st, log((double)n), (const double*)d_part, (int)nb,
                       lnZ, neff);
  rc = hipGetLastError() == hipSuccess ? RIFT_OK : RIFT_EDEVICE;
  // released in stream order, after the kernels above
  if (hipFreeAsync(space, st) != hipSuccess && !rc) rc = RIFT_EDEVICE;
  return rc;
}

}  // namespace
}  // namespace rift

extern "C" int rift_ile_wide_lnL(const rift_ile_point_wide* pt, int64_t n, const double* theta, double* lnL,
                                 void* stream) {
  if (!lnL && n > 0) return RIFT_EINVAL;
  return rift::wide_run(pt, n, theta, nullptr, lnL, nullptr, nullptr, stream);
}

extern "C" int rift_ile_wide_lnZ(const rift_ile_point_wide* pt, int64_t n, const double* theta, const double* lnw,
                                 double* lnZ, double* neff, double* lnL, void* stream) {
  if (!lnZ || n < 1) return RIFT_EINVAL;
  return rift::wide_run(pt, n, theta, lnw, lnL, lnZ, neff, stream);
}
