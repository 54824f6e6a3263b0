// The rules over polarisation, and over reference phase and polarisation
// together, on the coefficients that the likelihood kernel's data passes leave
// per sample:
//   q(u) = a + Re(c1 e^{iu}) + Re(c2 e^{2iu}),  u = 2 (psi' - psi).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/rift_ile.h"
#include "ile_angles.h"

namespace rift {
namespace {

constexpr double TWO_PI = 6.283185307179586477;
constexpr double PSI_LAPLACE_MIN_A = 100.0;
constexpr int PSI_FALLBACK_POINTS = 256;
constexpr int PSI_GRID = 32;  // points of the search for the dominant maximum

// Terms this far below the running maximum (nats) leave a double's sum of up
// to 1e7 terms as it is.
constexpr double FAR_BELOW = 60.0;

// q(u) and its first two derivatives.
__device__ __forceinline__ void psi_q(double a, double c1r, double c1i, double c2r, double c2i, double su, double cu,
                                      double* q, double* d1, double* d2) {
  const double s2 = 2.0 * su * cu, c2 = cu * cu - su * su;
  const double r1 = c1r * cu - c1i * su, i1 = c1r * su + c1i * cu;  // c1 e^{iu}
  const double r2 = c2r * c2 - c2i * s2, i2 = c2r * s2 + c2i * c2;  // c2 e^{2iu}
  *q = a + r1 + r2;
  *d1 = -i1 - 2.0 * i2;
  *d2 = -r1 - 4.0 * r2;
}

// tu [n][4] = cos u, sin u, cos 2u, sin 2u at u = 2 pi b / n.
__global__ void k_circle_table(int n, double* __restrict__ tu) {
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < n; b += gridDim.x * blockDim.x) {
    double s1, c1, s2, c2;
    sincospi(2.0 * (double)b / (double)n, &s1, &c1);
    sincospi(4.0 * (double)b / (double)n, &s2, &c2);
    tu[4 * b] = c1;
    tu[4 * b + 1] = s1;
    tu[4 * b + 2] = c2;
    tu[4 * b + 3] = s2;
  }
}

// Adds e^{q(u_b)} at the n points of the table to the running (max, sum).
// The points b and b + n/2 of an even n share q's even and odd parts.  Eight
// terms at a time: their largest first, one rescaling of the sum if it is a
// new maximum, then independent exponentials, skipped where all eight are far
// below (a chain of one running maximum per term serialised them).
__device__ __forceinline__ void circle_push(const RIFT_CONST double* tu, int n, double a, double c1r, double c1i,
                                            double c2r, double c2i, double& m, double& sum) {
  auto parts = [&](int b, double* e, double* o) {
    const RIFT_CONST double* U = tu + 4 * b;
    *o = fma(c1r, U[0], -c1i * U[1]);
    *e = fma(c2r, U[2], fma(-c2i, U[3], a));
  };
  auto raise = [&](double top) {
    if (top > m) {
      sum *= exp(m - top);  // 0 at the first terms
      m = top;
    }
  };
  int b = 0;
  const int pairs = (n & 1) ? 0 : n / 2;
  for (; b + 4 <= pairs; b += 4) {
    double e[4], o[4], top = -__builtin_inf();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      parts(b + j, &e[j], &o[j]);
      top = fmax(top, e[j] + fabs(o[j]));
    }
    raise(top);
    if (top >= m - FAR_BELOW) {
#pragma unroll
      for (int j = 0; j < 4; ++j) sum += exp(e[j] + o[j] - m) + exp(e[j] - o[j] - m);
    }
  }
  for (; b < pairs; ++b) {
    double e, o;
    parts(b, &e, &o);
    raise(e + fabs(o));
    sum += exp(e + o - m) + exp(e - o - m);
  }
  if (n & 1) {
    for (b = 0; b < n; ++b) {
      double e, o;
      parts(b, &e, &o);
      raise(e + o);
      sum += exp(e + o - m);
    }
  }
}

// The trapezoid and Laplace rules, a lane per sample.
__global__ void __launch_bounds__(256) k_psi(PsiRule G, int64_t cnt, const double* __restrict__ coef, int64_t stride,
                                             const double* __restrict__ tab, PsiOut out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  RIFT_GLOBAL double* value = as_global_w(out.L) + out.at(i);
  const RIFT_GLOBAL double* c = as_global(coef) + i;
  const double a = c[0], c1r = c[stride], c1i = c[2 * stride], c2r = c[3 * stride], c2i = c[4 * stride];
  const double flag = *value;
  const RIFT_CONST double* tu = as_const(tab);
  if (flag != flag) return;
  double q, d1, d2;
  int n = G.n;
  if (G.method == 1) {
    // the best of 32 equally spaced points, then Newton steps on q' = 0 (the
    // maximum is then the dominant one unless another lies within the grid's
    // resolution of it)
    constexpr int ST = PSI_FALLBACK_POINTS / PSI_GRID;
    double best = -__builtin_inf(), u = 0.0;
    for (int j = 0; j < PSI_GRID; ++j) {
      const RIFT_CONST double* U = tu + 4 * ST * j;
      const double v = a + (c1r * U[0] - c1i * U[1]) + (c2r * U[2] - c2i * U[3]);
      if (v > best) {
        best = v;
        u = TWO_PI * (double)j / PSI_GRID;
      }
    }
    for (int it = 0; it < 8; ++it) {
      double su, cu;
      sincos_many<1>(&u, &su, &cu);
      psi_q(a, c1r, c1i, c2r, c2i, su, cu, &q, &d1, &d2);
      if (!(d2 < 0.0)) break;
      u -= d1 / d2;
    }
    double su, cu;
    sincos_many<1>(&u, &su, &cu);
    psi_q(a, c1r, c1i, c2r, c2i, su, cu, &q, &d1, &d2);
    if (-d2 >= PSI_LAPLACE_MIN_A) {
      *value = q - 0.5 * log(TWO_PI * -d2);
      return;
    }
    n = PSI_FALLBACK_POINTS;
  }
  double m = -__builtin_inf(), sum = 0.0;
  circle_push(tu, n, a, c1r, c1i, c2r, c2i, m, sum);
  *value = m + log(sum) - log((double)n);
}

// ---------------------------------------------------------------------------
// The cell partition of Eq. (ap:psicells)
// ---------------------------------------------------------------------------
// With z = e^{iu}, 2 i z^2 q'(u) = 0 is the quartic
//   2 c2 z^4 + c1 z^3 - conj(c1) z - 2 conj(c2) = 0;
// its roots, by the Aberth-Ehrlich iteration, that lie within 1e-3 of the unit
// circle are polished by Newton's method on q'(u) and kept if they settle on a
// zero of q'.  Without c2, or with one below the rounding of c1 (the quartic's
// other two roots then lie near 0 and far out, beyond what the iteration's
// squares can hold), the two stationary points are closed forms.  The
// sorted angles cut the circle into cells on which q is monotone; each cell is
// integrated by 8-point Gauss-Legendre on sub-intervals of 2 sigma out to
// 8 sigma from its higher end, then of doubling length to its far end, sigma =
// min(A^{-1/2}, width / 8) from the curvature A = -q'' at that end.  A cell
// ends early where q, monotone in it, has fallen so far below the largest
// stationary value that nothing further on can count.  With fewer than two
// points found the circle is one cell, in which q need not be monotone: it is
// covered whole.
//
// A wavefront takes 64 samples: a lane per sample for the stationary points,
// then eight lanes per sample, one per node of a sub-interval.  Measured for 1e6
// prior samples at 3 detectors, 21 modes, SNR 600: 1.06 ms, and 0.25 ms for the
// data pass before it; with a lane per sample inside the data pass, 5.4 ms for both.
struct Cx {
  double x, y;
};
__device__ __forceinline__ Cx cx_mul(Cx a, Cx b) { return Cx{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ Cx cx_add(Cx a, Cx b) { return Cx{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Cx cx_sub(Cx a, Cx b) { return Cx{a.x - b.x, a.y - b.y}; }
// 1 / b, to a few units in the last place (the iteration corrects itself)
__device__ __forceinline__ Cx cx_inv(Cx b) {
  const double d = b.x * b.x + b.y * b.y;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  return Cx{b.x * r, -b.y * r};
}

constexpr int CELL_MAX = 4;
constexpr double C2_COUNTS = 1e-18;  // of c1: below it c2 moves neither a stationary point nor its value
constexpr double CELL_FAR = 50.0;  // nats below the largest value at which a cell ends
constexpr int CELL_STEPS = 1200;  // sub-intervals of a cell: doublings from the smallest sigma to a whole turn
struct CellPoint {
  double u, q, d2;
};

// The stationary angles in [0, 2 pi) with q and q'' there, sorted, the empty
// slots at +inf behind them.
__device__ __forceinline__ void psi_stationary(double a, double c1r, double c1i, double c2r, double c2i,
                                               CellPoint* st) {
#pragma unroll
  for (int k = 0; k < 4; ++k) st[k].u = __builtin_inf();
  const double scale = fmax(fmax(fabs(c1r), fabs(c1i)), 2.0 * fmax(fabs(c2r), fabs(c2i)));
  if (!(scale > 0.0)) return;
  double q, d1, d2, su, cu;
  if (2.0 * fmax(fabs(c2r), fabs(c2i)) <= C2_COUNTS * scale) {
    const double top = -atan2(c1i, c1r);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      double u = top + 3.14159265358979323846 * k;
      u = u < 0.0 ? u + TWO_PI : u;
      sincos_many<1>(&u, &su, &cu);
      psi_q(a, c1r, c1i, c2r, c2i, su, cu, &q, &d1, &d2);
      st[k] = CellPoint{u, q, d2};
    }
  } else {
    const Cx g1{c1r / scale, c1i / scale}, g2{2.0 * c2r / scale, 2.0 * c2i / scale};
    // e^{i (pi k / 2 + 0.4)}
    Cx z[4] = {Cx{0.92106099400288508, 0.38941834230865049}, Cx{-0.38941834230865049, 0.92106099400288508},
               Cx{-0.92106099400288508, -0.38941834230865049}, Cx{0.38941834230865049, -0.92106099400288508}};
    for (int it = 0; it < 60; ++it) {
      double moved = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // g2 z^4 + g1 z^3 - conj(g1) z - conj(g2) and its derivative
        Cx p = g2, dp = g2;
        p = cx_add(cx_mul(p, z[k]), g1);
        dp = cx_add(cx_mul(dp, z[k]), p);
        p = cx_mul(p, z[k]);
        dp = cx_add(cx_mul(dp, z[k]), p);
        p = cx_add(cx_mul(p, z[k]), Cx{-g1.x, g1.y});
        dp = cx_add(cx_mul(dp, z[k]), p);
        p = cx_add(cx_mul(p, z[k]), Cx{-g2.x, g2.y});
        if (p.x == 0.0 && p.y == 0.0) continue;
        const Cx ratio = cx_mul(p, cx_inv(dp));
        Cx sum{0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j != k) sum = cx_add(sum, cx_inv(cx_sub(z[k], z[j])));
        const Cx t = cx_mul(ratio, sum);
        const Cx w = cx_mul(ratio, cx_inv(Cx{1.0 - t.x, -t.y}));
        z[k] = cx_sub(z[k], w);
        moved = fmax(moved, fabs(w.x) + fabs(w.y));
      }
      if (!(moved > 1e-12)) break;  // Newton's method takes the rest
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double r2 = z[k].x * z[k].x + z[k].y * z[k].y;
      if (!(r2 >= 0.998001 && r2 <= 1.002001)) continue;
      double u = atan2(z[k].y, z[k].x);
      for (int it = 0; it < 30; ++it) {
        sincos_many<1>(&u, &su, &cu);
        psi_q(0.0, g1.x, g1.y, 0.5 * g2.x, 0.5 * g2.y, su, cu, &q, &d1, &d2);
        if (d2 == 0.0) break;
        const double step = d1 / d2;
        u -= step;
        if (fabs(step) < 1e-12) break;
      }
      sincos_many<1>(&u, &su, &cu);
      psi_q(0.0, g1.x, g1.y, 0.5 * g2.x, 0.5 * g2.y, su, cu, &q, &d1, &d2);
      if (!(fabs(d1) <= 1e-9)) continue;
      psi_q(a, c1r, c1i, c2r, c2i, su, cu, &q, &d1, &d2);
      u -= TWO_PI * floor(u / TWO_PI);
      u = u >= TWO_PI ? u - TWO_PI : u;
      st[k] = CellPoint{u, q, d2};
    }
  }
  auto order = [&](int x, int y) {
    if (st[y].u < st[x].u) {
      const CellPoint t = st[x];
      st[x] = st[y];
      st[y] = t;
    }
  };
  order(0, 1);
  order(2, 3);
  order(0, 2);
  order(1, 3);
  order(1, 2);
}

// A sample's cells as its eight lanes read them: the higher end, the direction
// away from it, the width, sigma, and q at the higher end.
struct CellLds {
  double c[5][64];                // a, c1, c2
  double m[64];                   // the largest value at an end
  double start[CELL_MAX][64], width[CELL_MAX][64], sigma[CELL_MAX][64], top[CELL_MAX][64];
  int64_t at[64];                 // where its value goes
  int32_t n[64], dir[64];         // cells; bit c: cell c runs downwards from its higher end
};

__constant__ double kGL8X[8] = {-0.96028985649753623168, -0.79666647741362673959, -0.52553240991632898582,
                                -0.18343464249564980494, 0.18343464249564980494,  0.52553240991632898582,
                                0.79666647741362673959,  0.96028985649753623168};
__constant__ double kGL8W[8] = {0.10122853629037625915, 0.22238103445337447054, 0.31370664587788728734,
                                0.36268378337836198297, 0.36268378337836198297, 0.31370664587788728734,
                                0.22238103445337447054, 0.10122853629037625915};

__global__ void __launch_bounds__(128) k_psi_cells(int64_t cnt, const double* __restrict__ coef, int64_t stride,
                                                   PsiOut out) {
  __shared__ CellLds lds[2];
  const int lane = threadIdx.x & 63;
  CellLds& S = lds[threadIdx.x >> 6];
  const int64_t base = (blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
  if (base >= cnt) return;
  {
    const int64_t i = base + lane < cnt ? base + lane : cnt - 1;
    const RIFT_GLOBAL double* p = as_global(coef) + i;
    const double a = p[0], c1r = p[stride], c1i = p[2 * stride], c2r = p[3 * stride], c2i = p[4 * stride];
    const int64_t o = out.at(i);
    const double flag = as_global(out.L)[o];
    const bool bad = flag != flag;
    S.at[lane] = o;
    S.c[0][lane] = a;
    S.c[1][lane] = c1r;
    S.c[2][lane] = c1i;
    S.c[3][lane] = c2r;
    S.c[4][lane] = c2i;
    int nc = 0, dir = 0;
    double m = 0.0;
    if (!bad) {
      CellPoint st[4];
      psi_stationary(a, c1r, c1i, c2r, c2i, st);
      // repeats (two roots settling on one point) leave
      int ns = st[0].u < __builtin_inf() ? 1 : 0;
      CellPoint pt[4] = {st[0], st[1], st[2], st[3]};
#pragma unroll
      for (int k = 1; k < 4; ++k) {
        const CellPoint prev = ns == 1 ? pt[0] : (ns == 2 ? pt[1] : pt[2]);
        if (st[k].u < __builtin_inf() && (ns == 0 || st[k].u - prev.u > 1e-12)) {
          if (ns == 1) pt[1] = st[k];
          else if (ns == 2) pt[2] = st[k];
          else pt[3] = st[k];
          ++ns;
        }
      }
      auto put = [&](int c, CellPoint lo, CellPoint hi) {
        const double width = hi.u - lo.u;
        const bool up = lo.q >= hi.q;  // the higher end is the lower angle
        const double A = -(up ? lo.d2 : hi.d2), top = up ? lo.q : hi.q;
        S.start[c][lane] = up ? lo.u : hi.u;
        S.width[c][lane] = width;
        S.sigma[c][lane] = A > 0.0 ? fmin(1.0 / sqrt(A), width / 8.0) : width / 8.0;
        S.top[c][lane] = top;
        if (!up) dir |= 1 << c;
        m = c == 0 ? top : fmax(m, top);
      };
      if (ns < 2) {
        double q, d1, d2;
        psi_q(a, c1r, c1i, c2r, c2i, 0.0, 1.0, &q, &d1, &d2);
        put(0, CellPoint{0.0, q, d2}, CellPoint{TWO_PI, q, d2});
        nc = 1;
      } else {
        nc = ns;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (c < ns) {
            CellPoint hi = c == 0 ? pt[1] : c == 1 ? pt[2] : pt[3];
            if (c + 1 == ns || c == 3) {
              hi = pt[0];
              hi.u += TWO_PI;
            }
            put(c, pt[c], hi);
          }
        }
      }
    }
    S.m[lane] = m;
    S.n[lane] = nc;
    S.dir[lane] = dir;
  }
  // the wavefront's own scratch: written before it is read
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int g = lane & 7;
  const double xg = 0.5 + 0.5 * kGL8X[g], wg = 0.5 * kGL8W[g];
  for (int r = 0; r < 8; ++r) {
    const int s = 8 * r + (lane >> 3);
    const double a = S.c[0][s], c1r = S.c[1][s], c1i = S.c[2][s], c2r = S.c[3][s], c2i = S.c[4][s];
    const double m0 = S.m[s];
    const int nc = S.n[s], dir = S.dir[s];
    double m = m0, sum = 0.0;
    int c = -1, j = 0;
    double start = 0.0, width = 0.0, sigma = 0.0, d0 = 0.0, sgn = 1.0;
    auto next = [&]() {
      do {
        ++c;
      } while (c < nc && S.top[c][s] < m0 - CELL_FAR);
      if (c < nc) {
        start = S.start[c][s];
        width = S.width[c][s];
        sigma = S.sigma[c][s];
        sgn = (dir >> c) & 1 ? -1.0 : 1.0;
      }
      d0 = 0.0;
      j = 1;
    };
    next();
    while (__any(c < nc)) {
      // every lane takes part (the far node's value is passed on); a finished
      // sample's lanes add nothing
      const bool on = c < nc;
      const double d1 = fmin(width, j <= 4 ? 2.0 * sigma * j : 2.0 * d0);
      const double h = d1 - d0;
      double su, cu, q, q1, q2;
      const double u = fma(sgn, fma(h, xg, d0), start);
      sincos_near<1>(&u, &su, &cu);
      psi_q(a, c1r, c1i, c2r, c2i, su, cu, &q, &q1, &q2);
      const double qfar = __shfl(q, lane | 7);
      if (on) {
        if (q > m) {  // only where a stationary point was not found
          sum *= exp(m - q);
          m = q;
        }
        sum = fma(h * wg, exp(q - m), sum);
        d0 = d1;
        ++j;
        if (!(d0 < width) || (nc > 1 && qfar < m0 - CELL_FAR) || j > CELL_STEPS) next();
      }
    }
    double mx = m;
#pragma unroll
    for (int o = 4; o >= 1; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (m != mx) sum *= exp(m - mx);
#pragma unroll
    for (int o = 4; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
    if (g == 0 && base + s < cnt && nc > 0) as_global_w(out.L)[S.at[s]] = mx + log(sum) - 1.8378770664093454836;  // ln 2 pi
  }
}

// ---------------------------------------------------------------------------
// The joint phiref / psi grid (ERAI)
// ---------------------------------------------------------------------------
// Tables: wd [n_phi][NDM] and wq [n_phi][NQM], the harmonics 1, cos alpha,
// sin alpha, .. at the grid's phases (zero past the harmonics in use).
__global__ void k_erai_tables(int n_phi, int nd, int nq, int NDM, int NQM, double* __restrict__ wd,
                              double* __restrict__ wq) {
  const int stride = gridDim.x * blockDim.x;
  auto harmonic = [&](int a, int j) {
    if (j == 0) return 1.0;
    const int m = (j + 1) / 2;
    const double x = 2.0 * (double)((int64_t)m * a % n_phi) / (double)n_phi;
    return j & 1 ? cospi(x) : sinpi(x);
  };
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n_phi * NDM; e += stride) {
    const int a = e / NDM, j = e - (e / NDM) * NDM;
    wd[e] = j < nd ? harmonic(a, j) : 0.0;
  }
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n_phi * NQM; e += stride) {
    const int a = e / NQM, j = e - (e / NQM) * NQM;
    wq[e] = j < nq ? harmonic(a, j) : 0.0;
  }
}

// One sample per lane, its harmonics in registers (zero past nd, nq); the grid
// loops are uniform, the tables read with uniform addresses.  Bound by the
// exponentials: 512 of them per sample on a 32 x 16 grid take 0.75 ms for 1e6
// samples (0.86 ms with one running maximum per term).
template <int NDM, int NQM>
__global__ void __launch_bounds__(256) k_erai(int64_t cnt, int nd, int nq, int n_phi, int n_psi,
                                              const double* __restrict__ ang, int64_t stride,
                                              const double* __restrict__ wd, const double* __restrict__ wq,
                                              const double* __restrict__ tu, double ln_scale, PsiOut out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  RIFT_GLOBAL double* value = as_global_w(out.L) + out.at(i);
  double c1r[NDM], c1i[NDM], ca[NQM], c2r[NQM], c2i[NQM];
  const RIFT_GLOBAL double* p = as_global(ang) + i;
#pragma unroll
  for (int j = 0; j < NDM; ++j) {
    c1r[j] = j < nd ? p[(int64_t)(2 * j) * stride] : 0.0;
    c1i[j] = j < nd ? p[(int64_t)(2 * j + 1) * stride] : 0.0;
  }
#pragma unroll
  for (int j = 0; j < NQM; ++j) {
    const int64_t r = 2 * nd + 3 * j;
    ca[j] = j < nq ? p[r * stride] : 0.0;
    c2r[j] = j < nq ? p[(r + 1) * stride] : 0.0;
    c2i[j] = j < nq ? p[(r + 2) * stride] : 0.0;
  }
  const double flag = *value;
  double m = -__builtin_inf(), sum = 0.0;
  for (int f = 0; f < n_phi; ++f) {
    const RIFT_CONST double* Wd = as_const(wd) + f * NDM;
    const RIFT_CONST double* Wq = as_const(wq) + f * NQM;
    double C1r = 0.0, C1i = 0.0, A = 0.0, C2r = 0.0, C2i = 0.0;
#pragma unroll
    for (int j = 0; j < NDM; ++j) {
      C1r = fma(Wd[j], c1r[j], C1r);
      C1i = fma(Wd[j], c1i[j], C1i);
    }
#pragma unroll
    for (int j = 0; j < NQM; ++j) {
      A = fma(Wq[j], ca[j], A);
      C2r = fma(Wq[j], c2r[j], C2r);
      C2i = fma(Wq[j], c2i[j], C2i);
    }
    circle_push(as_const(tu), n_psi, A, C1r, C1i, C2r, C2i, m, sum);
  }
  *value = (flag == flag && sum == sum) ? m + log(sum) + ln_scale : __builtin_nan("");
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
int launched() { return hipGetLastError() == hipSuccess ? RIFT_OK : RIFT_EDEVICE; }

int dm_of(int m_max) { return m_max <= 2 ? 5 : 9; }
int qm_of(int m_max) { return m_max <= 2 ? 9 : 17; }

}  // namespace

size_t psi_tables_len(const PsiRule& r) {
  return r.method == 2 ? 0 : 4 * (size_t)(r.method == 1 ? PSI_FALLBACK_POINTS : r.n);
}

int psi_tables(const PsiRule& r, double* tab, hipStream_t st) {
  if (r.method == 2) return RIFT_OK;
  const int n = r.method == 1 ? PSI_FALLBACK_POINTS : r.n;
  hipLaunchKernelGGL(k_circle_table, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, tab);
  return launched();
}

int run_psi(const PsiRule& r, int64_t cnt, const double* coef, int64_t stride, const double* tab,
            const PsiOut& out, hipStream_t st) {
  if ((cnt + 127) / 128 > 0x7fffffff) return RIFT_EUNSUPPORTED;
  if (r.method == 2)
    hipLaunchKernelGGL(k_psi_cells, dim3(blocks_for(cnt, 128)), dim3(128), 0, st, cnt, coef, stride, out);
  else
    hipLaunchKernelGGL(k_psi, dim3(blocks_for(cnt, 256)), dim3(256), 0, st, r, cnt, coef, stride, tab, out);
  return launched();
}

size_t erai_tables_len(int n_phi, int n_psi, int m_max) {
  return (size_t)n_phi * (dm_of(m_max) + qm_of(m_max)) + 4 * (size_t)n_psi;
}

int erai_tables(int n_phi, int n_psi, int m_max, double* tab, hipStream_t st) {
  const int NDM = dm_of(m_max), NQM = qm_of(m_max);
  double* wq = tab + (size_t)n_phi * NDM;
  hipLaunchKernelGGL(k_erai_tables, dim3(std::min(blocks_for((int64_t)n_phi * NQM, 256), 1024u)), dim3(256), 0, st,
                     n_phi, 2 * m_max + 1, 4 * m_max + 1, NDM, NQM, tab, wq);
  hipLaunchKernelGGL(k_circle_table, dim3(blocks_for(n_psi, 256)), dim3(256), 0, st, n_psi,
                     wq + (size_t)n_phi * NQM);
  return launched();
}

int run_erai(int64_t cnt, int n_phi, int n_psi, int m_max, const double* ang, int64_t stride, const double* tab,
             const PsiOut& out, hipStream_t st) {
  if ((cnt + 255) / 256 > 0x7fffffff) return RIFT_EUNSUPPORTED;
  const int nd = 2 * m_max + 1, nq = 4 * m_max + 1;
  const double* wq = tab + (size_t)n_phi * dm_of(m_max);
  const double* tu = wq + (size_t)n_phi * qm_of(m_max);
  const double ln_scale = -log((double)n_phi * (double)n_psi);
  const dim3 grid(blocks_for(cnt, 256)), block(256);
  if (m_max <= 2)
    hipLaunchKernelGGL((k_erai<5, 9>), grid, block, 0, st, cnt, nd, nq, n_phi, n_psi, ang, stride, tab, wq, tu, ln_scale,
                       out);
  else
    hipLaunchKernelGGL((k_erai<9, 17>), grid, block, 0, st, cnt, nd, nq, n_phi, n_psi, ang, stride, tab, wq, tu,
                       ln_scale, out);
  return launched();
}

}  // namespace rift
