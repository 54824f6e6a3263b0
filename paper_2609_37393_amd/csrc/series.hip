// The contracted series of the time marginals (see ile_series.h): the row
// contraction, the rules on the contracted rows, and the band rule's
// reconstruction between its nodes on the FP64 matrix cores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/rift_ile.h"
#include "ile_series.h"

namespace rift {
namespace {

constexpr int SERIES_GROUP = 256;  // samples a wavefront of k_series_rows looks through

// ---------------------------------------------------------------------------
// c_k[r] = Re sum_i conj(x F_k Y_i) Q_{k,i}[r]
// ---------------------------------------------------------------------------
// [samples x 2M][2M x rows] is a dense product in which a sample meets only
// the rows of its own window, so it runs on the FP64 matrix cores with the
// rows held still: a wavefront keeps 64 consecutive rows of one detector's
// table as B operands (NG doubles a lane and 16 rows), lists the samples of
// its group whose window meets them, and takes those 16 at a time as A.  Both
// operands put element q NG + b of the 4 NG-long inner dimension at quad q of
// step b, so a lane reads NG consecutive doubles of its sample.
template <int NG>
__global__ void __launch_bounds__(256) k_series_rows(SeriesArgs a) {
  typedef double D4 __attribute__((ext_vector_type(4)));
  __shared__ uint16_t list[4][SERIES_GROUP];
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
  const int wave = threadIdx.x >> 6;
  const int tile = __builtin_amdgcn_readfirstlane(a.tile0 + (int)(blockIdx.x * 4) + wave);
  PDesc P = as_const(a.P);
  const int K = P->K, NR = P->n_t + 2 * QPAD, W2 = 2 * P->w64, sh = P->w64 == QW64 ? 4 : 2, NGR = q_groups(P->M, P->w64);
  const int lo = tile * 64;
  if (lo >= NR) return;
  const int k = blockIdx.y;
  // the samples whose window [r, r + wn) meets rows lo .. lo + 63
  const int s0 = blockIdx.z * SERIES_GROUP, s1 = s0 + SERIES_GROUP < a.cnt ? s0 + SERIES_GROUP : a.cnt;
  const RIFT_GLOBAL int32_t* r0 = as_global(a.r0) + (int64_t)k * a.cs + a.off;
  int count = 0;
  for (int sb = s0; sb < s1; sb += 64) {
    const int s = sb + lane;
    const int r = s < s1 ? r0[s] : 0x3fffffff;
    const bool meets = r <= lo + 63 && r + a.wn > lo;
    const uint64_t mask = __ballot(meets);
    const int at = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (meets) list[wave][count + at] = (uint16_t)(s - s0);
    count += __builtin_popcountll(mask);
  }
  if (count == 0) return;
  // the wavefront's own list: written before it is read
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // B: element e of row lo + 16 t + col (mode e / 2, part e & 1).  The products'
  // steps take the elements in pairs, so that a quad reads 16 bytes at a time
  // and the four of a row 64 (58 us for a chunk's rows of 21 modes; 63 with NG
  // elements in a run per quad).
  auto element = [&](int b) { return b < NG / 2 * 2 ? 8 * (b / 2) + 2 * quad + (b & 1) : 4 * (NG - 1) + quad; };
  double B[4][NG];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = lo + 16 * t + col;
    const RIFT_GLOBAL double* Q =
        as_global(P->Q64) + W2 * ((int64_t)k * NGR * NR + (row < NR ? row : NR - 1));
#pragma unroll
    for (int b = 0; b < NG; ++b) {
      const int e = element(b), grp = e >> sh;
      B[t][b] = grp < NGR ? Q[W2 * (int64_t)grp * NR + (e & (W2 - 1))] : 0.0;
    }
  }
  double A[NG];
  auto load = [&](int j, int* s, int* r) {
    *s = s0 + list[wave][j < count ? j : count - 1];
    *r = r0[*s];
    const RIFT_GLOBAL double* c = as_global(a.coef) + ((int64_t)(a.off + *s) * K + k) * series_coef_len(NG);
#pragma unroll
    for (int b = 0; b < NG; ++b) A[b] = c[element(b)];
  };
  int s, rs;
  load(col, &s, &rs);
  for (int j = 0; j < count; j += 16) {
    D4 d[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = D4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < NG; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) d[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[b], B[t][b], d[t], 0, 0, 0);
    const int cur = s, rc = rs;
    if (j + 16 < count) load(j + 16 + col, &s, &rs);
    // lane: samples 4 r + quad, row lo + 16 t + col
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int sr = __shfl(cur, 4 * r + quad);
      const bool in = j + 4 * r + quad < count;
      const int i0 = lo + col - __shfl(rc, 4 * r + quad);
      RIFT_GLOBAL double* o = as_global_w(a.c) + ((int64_t)sr * K + k) * a.wp;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int idx = i0 + 16 * t;
        if (in && idx >= 0 && idx < a.wn) o[idx] = d[t][r];
      }
    }
  }
}

// x kappa(t) of one sample from its contracted rows (sample and detector
// uniform, the time per lane).
template <int KT>
struct SeriesRead {
  double pt0, inv_dt;
  int n_t, K, wn;
  int r0[KT];
  double delay[KT];
  const RIFT_GLOBAL double* c[KT];
  __device__ __forceinline__ SeriesRead(const SeriesArgs& a, int s) {
    PDesc P = as_const(a.P);
    pt0 = P->t0;
    inv_dt = P->inv_dt;
    n_t = P->n_t;
    K = P->K;
    wn = a.wn;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      if (k >= K) break;
      r0[k] = as_const(a.r0)[(int64_t)k * a.cs + a.off + s];
      delay[k] = as_const(a.delay)[(int64_t)k * a.cs + a.off + s];
      c[k] = as_global(a.c) + ((int64_t)s * K + k) * a.wp;
    }
  }
  __device__ __forceinline__ double at(double t) const {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      if (k >= K) break;
      double f, w[4];
      bool bad = false;
      int i = series_row(t - delay[k], pt0, inv_dt, n_t, &f, &bad) - r0[k];
      i = i < 0 ? 0 : (i > wn - 4 ? wn - 4 : i);
      lagrange4(f, w);
      const RIFT_GLOBAL double* p = c[k] + i;
      v = fma(w[3], p[3], fma(w[2], p[2], fma(w[1], p[1], fma(w[0], p[0], v))));
    }
    return v;
  }
};

// e^{-746} and below is zero in FP64: a term that far below the running
// maximum leaves the sum as it is.
constexpr double EXP_ZERO = 746.0;

// Adds e^l to the running (max, sum).  At high amplitude nearly every term is
// a zero, and a wavefront that holds none but zeros branches past the
// exponential.  A NaN poisons the sum.
__device__ __forceinline__ void lse_push(double l, double& m, double& sum) {
  if (!(l < m - EXP_ZERO)) {
    const double d = l - m;
    const double e = exp(-fabs(d));
    const bool up = d > 0.0;
    sum = up ? fma(sum, e, 1.0) : sum + e;
    m = up ? l : m;
  }
}

// A wavefront per sample, its lanes over the times.  Bound by reading the
// contracted rows (each once from memory, the taps' overlaps from the vector
// cache).
template <int KT>
__global__ void __launch_bounds__(256) k_series_simpson(SeriesArgs a, TimeRule T, double* __restrict__ L) {
  const int lane = threadIdx.x & 63;
  const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (s >= a.cnt) return;
  const SeriesRead<KT> S(a, s);
  const double base = as_const(a.base)[a.off + s];
  double m = -__builtin_inf(), sum = 0.0;
  for (int k = lane; k < T.n; k += 64) {
    const double lw = (k == 0 || k == T.n - 1) ? T.lw_end : ((k & 1) ? T.lw_odd : T.lw_even);
    lse_push(S.at(fma((double)k, T.h, T.t0)) + base + lw, m, sum);
  }
  const double mx = dmax_wave(m);
  sum = dsum_wave(sum == 0.0 ? 0.0 : sum * exp(m - mx));
  if (lane == 0) as_global_w(L)[a.i0 + a.off + s] = sum == sum ? mx + log(sum) + T.ln_scale : __builtin_nan("");
}

// The band rule's node values y[s][NB] (zero past n), a lane per node, and
// the time-independent remainder in place of the result.
template <int KT>
__global__ void __launch_bounds__(256) k_series_nodes(SeriesArgs a, int nb, double* __restrict__ y,
                                                      double* __restrict__ L) {
  const int lane = threadIdx.x & 63;
  const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (s >= a.cnt) return;
  const SeriesRead<KT> S(a, s);
  if (lane < nb) {
    const double v = S.at(fma((double)lane, a.h, a.t0));
    as_global_w(y)[(int64_t)(a.off + s) * nb + lane] = lane < a.n ? v : 0.0;
  }
  if (lane == 0) as_global_w(L)[a.i0 + a.off + s] = as_const(a.base)[a.off + s];
}

// ---------------------------------------------------------------------------
// The band rule between the nodes (Eq. (ap:tband))
// ---------------------------------------------------------------------------
// The sinc series from the nodes to the fine points mirrors: node n - 1 - j
// reaches fine point last - k as node j reaches k.  So the sum and the
// difference of the values at k and last - k are the products of the halves
//   e_j = (y_j + y_{n-1-j}) / 2,  o_j = (y_j - y_{n-1-j}) / 2,  j < ceil(n/2)
// (e of an odd n's middle node is y/2) with sinc(k/M - j) +- sinc(k/M - (n-1-j)):
// half the multiply-adds, over k <= last / 2.
// S[0][j][k], S[1][j][k]: the sum and the difference for j < NB/2 and k < FP
// (both padded; zero past ceil(n/2)).  sin(pi (d + f)) = (-1)^d sin(pi f):
// exact zeros at the nodes.
__global__ void k_sinc_matrix(int hb, int n, int M, int fp, double* __restrict__ S) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= fp) return;
  const int ii = k / M, s = k - ii * M;
  const double f = (double)s / (double)M;
  const double sp = sinpi(f);
  auto sinc = [&](int j) {
    const int d = ii - j;
    if (s == 0) return d == 0 ? 1.0 : 0.0;
    return ((d & 1) ? -1.0 : 1.0) * sp / (3.14159265358979323846 * ((double)d + f));
  };
  for (int j = blockIdx.y; j < hb; j += gridDim.y) {
    const bool in = j < (n + 1) / 2;
    const double u = in ? sinc(j) : 0.0, v = in ? sinc(n - 1 - j) : 0.0;
    S[(int64_t)j * fp + k] = u + v;
    S[(int64_t)(hb + j) * fp + k] = u - v;
  }
}

// ln L_t = ln[(1 / ((n - 1) M)) sum_k w_k e^{l_k}], w = 1, ends 1/2, of the
// values l_k = x kappa(t_k) + base: [samples x nodes][nodes x fine] is a dense
// product, so it runs on the FP64 matrix cores (16 x 16 x 4 tiles: lane l
// holds A[l & 15][l >> 4], B[l >> 4][l & 15] and D[4 r + (l >> 4)][l & 15],
// r < 4).  A wavefront keeps 16 samples' halves (NB / 4 doubles a lane) and
// walks the fine points 16 at a time; the four wavefronts of a block read the
// same columns of S.  L holds the remainder on entry, ln L_t on return.
template <int NB>
__global__ void __launch_bounds__(256) k_band(int64_t cnt, int n, int M, int fp, const double* __restrict__ y,
                                              int64_t ys, int64_t yj, const double* __restrict__ S, double ln_scale,
                                              double* __restrict__ L) {
  typedef double D4 __attribute__((ext_vector_type(4)));
  constexpr int KB = NB / 8;  // steps of four halves
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
  const int64_t i0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  const int64_t ia = i0 + col < cnt ? i0 + col : cnt - 1;
  double e[KB], o[KB];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int j = 4 * b + quad, jm = n - 1 - j;
    const RIFT_GLOBAL double* yi = as_global(y) + ia * ys;
    const double u = j <= jm ? 0.5 * yi[j * yj] : 0.0, v = j <= jm ? 0.5 * yi[jm * yj] : 0.0;
    e[b] = j == jm ? u : u + v;
    o[b] = u - v;
  }
  double base[4], m[4], sum[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = i0 + 4 * r + quad;
    base[r] = i < cnt ? as_global(L)[i] : 0.0;
    m[r] = -__builtin_inf();
    sum[r] = 0.0;
  }
  const int last = (n - 1) * M;
  const RIFT_GLOBAL double* Be = as_global(S) + (int64_t)quad * fp + col;
  const RIFT_GLOBAL double* Bo = Be + (int64_t)(NB / 2) * fp;
  double be[KB], bo[KB];
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    be[b] = Be[(int64_t)4 * b * fp];
    bo[b] = Bo[(int64_t)4 * b * fp];
  }
  for (int f = 0; 2 * f <= last; f += 16) {
    D4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      E = __builtin_amdgcn_mfma_f64_16x16x4f64(e[b], be[b], E, 0, 0, 0);
      O = __builtin_amdgcn_mfma_f64_16x16x4f64(o[b], bo[b], O, 0, 0, 0);
    }
    // the next columns are on their way while this tile's exponentials run
    const int fn = 2 * (f + 16) <= last ? f + 16 : f;
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      be[b] = Be[(int64_t)4 * b * fp + fn];
      bo[b] = Bo[(int64_t)4 * b * fp + fn];
    }
    const int k = f + col;
    const double lw = k == 0 ? -0.69314718055994530942 : 0.0;  // both ends
    if (2 * k <= last) {
#pragma unroll
      for (int r = 0; r < 4; ++r) lse_push(E[r] + O[r] + base[r] + lw, m[r], sum[r]);
      if (2 * k < last) {
#pragma unroll
        for (int r = 0; r < 4; ++r) lse_push(E[r] - O[r] + base[r] + lw, m[r], sum[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double mx = m[r];
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1) mx = fmax(mx, __shfl_xor(mx, s));
    double v = sum[r] == 0.0 ? 0.0 : sum[r] * exp(m[r] - mx);
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1) v += __shfl_xor(v, s);
    const int64_t i = i0 + 4 * r + quad;
    if (col == 0 && i < cnt) as_global_w(L)[i] = v == v ? mx + log(v) + ln_scale : __builtin_nan("");
  }
}

// The instance of the row contraction: one for every count of mode pairs, so that
// none pays for another's products (3 detectors, 1e5 samples, 41 and 601 times, us:
// the complete l <= 3 set of 12 modes 213 and 1041, by the instance of 16 modes 249
// and 1095; 7 modes 180, 994 against 199, 1014 by that of 9; 17 modes 268, 1159
// against 292, 1252 by that of 21), but for 12 pairs, which run as 13 (23 modes 583
// and 1769, by its own 555 and 1806; 3e4 samples 220, 555 against 220, 572).
int series_groups(int M) {
  const int g = (M + 1) / 2;
  return g == 12 ? 13 : g;
}
static_assert((MMAX + 1) / 2 <= 13, "the largest instance holds every mode");

// Workspace of a run: the samples' coefficients (and node values) of one
// outer chunk, and the contracted rows of one inner chunk.
constexpr size_t SERIES_WS_OUT = (size_t)112 << 20;
constexpr size_t SERIES_WS_ROWS = (size_t)112 << 20;

int window_rows(const PointDesc& D, double h, int n) {
  const double span = (double)(n - 1) * h * D.inv_dt;
  const int all = D.n_t + 2 * QPAD;
  return span < (double)all ? std::min(all, (int)span + 8) : all;
}

struct Layout {
  int ng, wn, wp, nb;
  size_t per_out, per_rows;  // bytes per sample
  int64_t outer, inner;      // samples of the chunks
  size_t bytes() const { return (size_t)outer * per_out + (size_t)inner * per_rows; }
};
Layout layout(const PointDesc& D, double h, int n, bool band) {
  Layout l;
  l.ng = series_groups(D.M);
  l.wn = window_rows(D, h, n);
  l.wp = (l.wn + 15) / 16 * 16;
  l.nb = band ? band_pad(n) : 0;
  l.per_out = sizeof(double) * ((size_t)D.K * (series_coef_len(l.ng) + 1) + 1 + l.nb) + sizeof(int32_t) * D.K;
  l.per_rows = sizeof(double) * (size_t)D.K * l.wp;
  auto chunk = [&](size_t cap, size_t per) {
    const int64_t fit = std::max<int64_t>(64, (int64_t)(cap / per) / 64 * 64);
    return std::min<int64_t>(fit, (D.n + 63) / 64 * 64);
  };
  l.outer = chunk(SERIES_WS_OUT, l.per_out);
  l.inner = std::min(chunk(SERIES_WS_ROWS, l.per_rows), l.outer);
  return l;
}

}  // namespace

bool series_holds(const PointDesc& D, double t0, double h, int n) {
  // times so large that a row's own rounding is not small against a row: the
  // windows' ends would not bound the rows between them
  const double big = std::max(std::max(fabs(t0), fabs(t0 + (n - 1) * h)), fabs(D.t0)) + 1.0;
  return big * D.inv_dt < 1.0e12;
}

// The two estimates (us) are fits to 321 calls of 1 to 1e5 samples a point, 1 to 64
// points, 1 to 8 detectors, 2 to 21 modes, 2 to 301 times 1 to 30 rows apart,
// each timed both ways; they hold to 20 - 30%, and the choice costs a hundredth on
// average and 1.4 times at worst over those calls.  A launch of tiles whose blocks
// leave the chip idle runs its times one after the other; the contraction takes
// tiles of 64 rows, a launch sequence per point, and writes and reads the rows it
// keeps.
// Measured, contracted against per time: 21 modes x 3 detectors, 1e5 samples, 41
// times 1, 4, 12 rows apart 352, 485, 1018 against 922; 2 x 3, 1e5, 41 times
// 128, 213, 590 against 121, 101 times 201 against 274; 3 times of 5e4 samples of 9
// x 3 104 against 34; 64 points of 1000 samples, 2 x 3, 41 times 1529 against 112.
double series_us(const PointDesc& D, double h, int n) {
  const double wn = window_rows(D, h, n), tiles = wn + 63.0, ng = series_groups(D.M), K = D.K;
  return 22.0 + 0.73 * K * ng +
         1e-5 * (double)D.n * K * (std::max(0.039 * tiles * ng, 0.233 * tiles) + 5.1 * ng + 0.204 * wn);
}
double time_step_us(const PointDesc& D) { return 0.6 + 0.167 * D.K * (q_groups(D.M, D.w64) * D.w64); }

size_t series_bytes(const PointDesc& D, double h, int n, bool band) { return layout(D, h, n, band).bytes(); }

int band_pad(int n) { return n <= 16 ? 16 : (n <= 32 ? 32 : 64); }
static int fine_pad(int n, int fine) { return ((n - 1) * fine / 2 + 1 + 15) / 16 * 16; }
size_t sinc_matrix_len(int n, int fine) { return (size_t)band_pad(n) * fine_pad(n, fine); }

int sinc_matrix(int n, int fine, double* S, hipStream_t st) {
  const int fp = fine_pad(n, fine), nb = band_pad(n);
  hipLaunchKernelGGL(k_sinc_matrix, dim3((fp + 255) / 256, nb / 2), dim3(256), 0, st, nb / 2, n, fine, fp, S);
  return hipGetLastError() == hipSuccess ? RIFT_OK : RIFT_EDEVICE;
}

int band_reconstruct(int64_t cnt, int n, int fine, const double* y, int64_t ys, int64_t yj, const double* S, double* L,
                     hipStream_t st) {
  const int nb = band_pad(n), fp = fine_pad(n, fine);
  const double ln_scale = -log((double)(n - 1) * (double)fine);
  const int64_t blocks = (cnt + 63) / 64;
  if (blocks > 0x7fffffff) return RIFT_EUNSUPPORTED;
  const dim3 grid((unsigned)blocks), block(256);
  if (nb == 16)
    hipLaunchKernelGGL(k_band<16>, grid, block, 0, st, cnt, n, fine, fp, y, ys, yj, S, ln_scale, L);
  else if (nb == 32)
    hipLaunchKernelGGL(k_band<32>, grid, block, 0, st, cnt, n, fine, fp, y, ys, yj, S, ln_scale, L);
  else
    hipLaunchKernelGGL(k_band<64>, grid, block, 0, st, cnt, n, fine, fp, y, ys, yj, S, ln_scale, L);
  return hipGetLastError() == hipSuccess ? RIFT_OK : RIFT_EDEVICE;
}

int run_series(const SeriesJob& j, hipStream_t st) {
  const PointDesc& D = *j.h_desc;
  const bool band = j.fine > 0;
  const Layout l = layout(D, j.tm.h, j.tm.n, band);
  const int K = D.K, KT = j.KT;
  if (j.ws_bytes < l.bytes()) return RIFT_EINVAL;
  SeriesArgs a{};
  a.P = j.d_desc;
  a.theta = j.theta;
  a.N = j.N;
  a.cs = (int32_t)l.outer;
  a.ng = l.ng;
  a.wn = l.wn;
  a.wp = l.wp;
  a.n = j.tm.n;
  a.t0 = j.tm.t0;
  a.h = j.tm.h;
  double* w = (double*)j.ws;
  a.c = w;
  w += (size_t)l.inner * K * l.wp;
  a.coef = w;
  w += (size_t)l.outer * K * series_coef_len(l.ng);
  double* y = w;
  w += (size_t)l.outer * l.nb;
  a.delay = w;
  w += (size_t)l.outer * K;
  a.base = w;
  w += l.outer;
  a.r0 = (int32_t*)w;
  series_coef_fn f = KT == 2 ? get_series_kt2(D.L) : KT == 3 ? get_series_kt3(D.L) : KT == 5 ? get_series_kt5(D.L)
                                                                                             : get_series_kt8(D.L);
  if (!f) return RIFT_EUNSUPPORTED;
  const size_t trig = D.L == 8 ? sizeof(double) * 34 * 128 : 0;
  // the tiles of 64 rows that some window can meet: delays lie within the
  // detectors' distances from the geocentre
  double far = 0.0;
  for (int k = 0; k < K; ++k)
    far = std::max(far, sqrt(D.rpos[k][0] * D.rpos[k][0] + D.rpos[k][1] * D.rpos[k][1] + D.rpos[k][2] * D.rpos[k][2]));
  const int rows = D.n_t + 2 * QPAD;
  auto row_of = [&](double t) { return std::min(std::max((t - D.t0) * D.inv_dt + QPAD, 0.0), (double)rows); };
  const int first = std::max(0, (int)row_of(j.tm.t0 - far * (1.0 + 1e-12)) - 4) / 64;
  const int end = std::min(rows, (int)row_of(j.tm.t0 + (j.tm.n - 1) * j.tm.h + far * (1.0 + 1e-12)) + 8);
  a.tile0 = first;
  const unsigned tiles = (unsigned)((end - 64 * first + 255) / 256);
  for (int64_t so = 0; so < D.n; so += l.outer) {
    a.i0 = D.s0 + so;
    const int no = (int)std::min<int64_t>(l.outer, D.n - so);
    a.off = 0;
    a.cnt = no;
    hipLaunchKernelGGL(f, dim3((unsigned)((no + 127) / 128)), dim3(128), trig, st, a);
    for (int si = 0; si < no; si += (int)l.inner) {
      a.off = si;
      a.cnt = (int)std::min<int64_t>(l.inner, no - si);
      const dim3 grid(tiles, (unsigned)K, (unsigned)((a.cnt + SERIES_GROUP - 1) / SERIES_GROUP));
      switch (l.ng) {
#define RIFT_ROWS(G) \
  case G: hipLaunchKernelGGL(k_series_rows<G>, grid, dim3(256), 0, st, a); break;
        RIFT_ROWS(1)
        RIFT_ROWS(2)
        RIFT_ROWS(3)
        RIFT_ROWS(4)
        RIFT_ROWS(5)
        RIFT_ROWS(6)
        RIFT_ROWS(7)
        RIFT_ROWS(8)
        RIFT_ROWS(9)
        RIFT_ROWS(10)
        RIFT_ROWS(11)
        RIFT_ROWS(13)
#undef RIFT_ROWS
      }
      const dim3 per4((unsigned)((a.cnt + 3) / 4));
#define RIFT_RULE(T)                                                                  \
  {                                                                                   \
    if (band)                                                                         \
      hipLaunchKernelGGL(k_series_nodes<T>, per4, dim3(256), 0, st, a, l.nb, y, j.L); \
    else                                                                              \
      hipLaunchKernelGGL(k_series_simpson<T>, per4, dim3(256), 0, st, a, j.tm, j.L);  \
  }
      if (KT == 2) RIFT_RULE(2)
      else if (KT == 3) RIFT_RULE(3)
      else if (KT == 5) RIFT_RULE(5)
      else RIFT_RULE(8)
#undef RIFT_RULE
      if (hipGetLastError() != hipSuccess) return RIFT_EDEVICE;
    }
    if (band) {
      const int rc = band_reconstruct(no, j.tm.n, j.fine, y, l.nb, 1, j.sinc, j.L + a.i0, st);
      if (rc) return rc;
    }
  }
  return RIFT_OK;
}

}  // namespace rift
