// The time marginals by contracted series.
//
// At fixed other parameters the data term at geocentric time t is
//   x kappa(t) = sum_k sum_tap w_tap(t) c_k[row_k(t) + tap],
//   c_k[r] = Re sum_i conj(x F_k Y_i) Q_{k,i}[r]:
// the modes are contracted once per table row of a detector's window instead
// of once per tap of every time.  Neighbouring times share rows, so a rule
// whose times lie closer than a few rows needs a fraction of the per-time
// form's work, and a row of Q is read by whole wavefronts (consecutive lanes,
// consecutive rows) instead of by a gather at every lane's own place.
//
// 3 detectors, 21 modes, 1e5 samples: 657 times at the table's spacing take
// 1.43 ms (per time 16.4 ms), of which the contraction 0.8 ms (three times its
// matrix-core time; 1.6 GB written), the rule's reads of it 0.5 ms; the band
// rule on 64 nodes with 16 fine intervals 1.39 ms (2.2 ms), of which its
// reconstruction 0.34 ms.  Where few times share a row, series_us and
// time_step_us decide for the per-time form.
//
// Per chunk of samples, with every array in one workspace:
//   k_series_coef    a lane per sample: x F_k Y_i, the delays, the first row
//                    of every detector's window, and -x^2 quad;
//   k_series_rows    the contraction, 64 rows of one detector per wavefront
//                    (this and the next in inner chunks, so that the rows are
//                    read back while they are in cache);
//   k_series_simpson or k_series_nodes
//                    a wavefront per sample: the taps at every time, then the
//                    Simpson rule's log-sum or the values at the band rule's
//                    nodes.
#pragma once

#include "ile_device.h"

namespace rift {

// Doubles per (sample, detector) of the coefficients, NG groups of two modes.
__host__ __device__ constexpr int series_coef_len(int NG) { return 4 * NG; }

struct SeriesArgs {
  const PointDesc* P;
  const double* theta;  // [7][N]
  int64_t N;
  int64_t i0;           // first column of the outer chunk (the coefficients')
  int32_t off;          // first sample of the launch within it
  int32_t cnt;          // samples of the launch
  int32_t cs;           // stride of the [K][cs] arrays
  int32_t ng;           // mode groups of the coefficients (>= ceil(M / 2))
  int32_t wn;           // rows kept of every window
  int32_t wp;           // their stride
  int32_t tile0;        // first tile of 64 rows that a window can meet
  int32_t n;            // times t0 + k h
  double t0, h;
  double* coef;         // [cs][K][4 ng]: x F Y of the internal modes, (re, im)
  int32_t* r0;          // [K][cs]: first (padded) row of the window
  double* delay;        // [K][cs]: r_k . N, so t_k = t - delay
  double* base;         // [cs]: -x^2 quad, NaN for a poisoned sample
  double* c;            // [cnt][K][wp]: the contracted rows of this launch's samples
};

// Padded first stencil row and cell fraction at arrival time tk (the
// arithmetic of sky_stencils).
__device__ __forceinline__ int series_row(double tk, double pt0, double inv_dt, int n_t, double* s, bool* bad) {
  double u = (tk - pt0) * inv_dt;
  if (!stencil_u(u, n_t)) *bad = true;
  const double jf = floor(u);
  if (s) *s = u - jf;
  int j0 = (int)jf - 1;
  j0 = j0 < -QPAD ? -QPAD : (j0 > n_t ? n_t : j0);
  return j0 + QPAD;
}

// A lane per sample.  Bound by its stores (4 ng doubles per detector, a lane's
// own 16-byte pieces) and the model norm's contraction; both are small beside
// the row contraction that follows.
template <int KT, int L>
__global__ void __launch_bounds__(128) k_series_coef(SeriesArgs a) {
  constexpr int NY = Cls<L>::NY;
  extern __shared__ __align__(16) unsigned char smem[];
  double* trig = reinterpret_cast<double*>(smem) + threadIdx.x;  // l <= 8 class only
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = s < a.cnt;
  const int64_t i = a.i0 + (live ? s : a.cnt - 1);
  PDesc P = opaque(a.P);
  const RIFT_GLOBAL double* th = as_global(a.theta) + i;
  const int64_t N = a.N;
  const double dist = th[6 * N];
  Sky<double, KT> S;
  double si, ci, sf, cf;
  sky_eval<double, KT, false>(P, th[0], th[N], th[2 * N], th[3 * N], th[4 * N], 0.0, S, si, ci, sf, cf);
  double cn[NY], sn[NY];
  incl_harmonics<double, NY>(ci, si, cn, sn);
  double wq = 0.0;
  const double quad = quad_term<double, KT, L, false>(P, trig, blockDim.x, ci, si, cf, sf, S.Fre, S.Fim, &wq);
  const double x = P->d_ref / dist;
  const double base = -x * x * quad;
  bool bad = !(fabs(x) <= 1.0e300) || !(fabs(base) <= 1.0e300);
  const int K = P->K, M = P->M, n_t = P->n_t;
  const double tl = fma((double)(a.n - 1), a.h, a.t0);
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    if (k >= K) break;
    const RIFT_CONST double* r = P->rpos[k];
    const double d = r[0] * S.N[0] + r[1] * S.N[1] + r[2] * S.N[2];
    // the arrival time is monotone in the rule's time, so finite ends make
    // every time finite and the rows of all times lie between the ends'
    const int row = series_row(a.t0 - d, P->t0, P->inv_dt, n_t, nullptr, &bad);
    (void)series_row(tl - d, P->t0, P->inv_dt, n_t, nullptr, &bad);
    if (live) {
      as_global_w(a.r0)[(int64_t)k * a.cs + s] = row;
      as_global_w(a.delay)[(int64_t)k * a.cs + s] = d;
    }
  }
  if (live) as_global_w(a.base)[s] = bad ? __builtin_nan("") : base;
  // Y_i = d_i(incl) e^{i m_i phi}, modes sorted by m
  C2<double> ph;
  ph.x = 1.0;
  ph.y = 0.0;
  const int mmin = P->m_min;
  for (int t = 0; t < -mmin; ++t) phase_down(ph, cf, sf);
  int mc = mmin < 0 ? mmin : 0;
  const int len = series_coef_len(a.ng);
  RIFT_GLOBAL double* co = as_global_w(a.coef) + (int64_t)(live ? s : 0) * K * len;
  for (int m = 0; m < 2 * a.ng; ++m) {
    double yx = 0.0, yy = 0.0;
    if (m < M) {
      const int mi = P->m[m];
      while (mc < mi) {
        phase_up(ph, cf, sf);
        ++mc;
      }
      const double dd = x * mode_d<double, NY>(P, m, cn, sn);
      yx = dd * ph.x;
      yy = dd * ph.y;
    }
    if (!live) continue;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      if (k >= K) break;
      co[k * len + 2 * m] = S.Fre[k] * yx - S.Fim[k] * yy;
      co[k * len + 2 * m + 1] = S.Fre[k] * yy + S.Fim[k] * yx;
    }
  }
}

typedef void (*series_coef_fn)(SeriesArgs);
series_coef_fn get_series_kt2(int L);
series_coef_fn get_series_kt3(int L);
series_coef_fn get_series_kt5(int L);
series_coef_fn get_series_kt8(int L);

// ---------------------------------------------------------------------------
// Host side (series.hip)
// ---------------------------------------------------------------------------
struct SeriesJob {
  const PointDesc* d_desc;  // the point, device and host copies
  const PointDesc* h_desc;
  int KT;
  const double* theta;
  int64_t N;
  TimeRule tm;              // times t0 + k h; Simpson weights (Simpson rule)
  int fine;                 // > 0: the band rule with `fine` intervals per node interval
  const double* sinc;       // band rule: the sinc matrix of sinc_matrix()
  double* L;                // [N] results
  void* ws;                 // workspace of series_bytes()
  size_t ws_bytes;
};
// Whether a point's rule can run by contracted series; what that costs a point, and
// one time of the per-time form on a lane (both us).
bool series_holds(const PointDesc& D, double t0, double h, int n);
double series_us(const PointDesc& D, double h, int n);
double time_step_us(const PointDesc& D);
// Workspace of a point's run (bounded; larger batches run in chunks).
size_t series_bytes(const PointDesc& D, double h, int n, bool band);
int run_series(const SeriesJob& j, hipStream_t st);

// The band rule's reconstruction after the node values: see series.hip.
int band_pad(int n);                       // padded node count
size_t sinc_matrix_len(int n, int fine);   // doubles of the matrix
int sinc_matrix(int n, int fine, double* S, hipStream_t st);
int band_reconstruct(int64_t cnt, int n, int fine, const double* y, int64_t ys, int64_t yj, const double* S, double* L,
                     hipStream_t st);

}  // namespace rift
