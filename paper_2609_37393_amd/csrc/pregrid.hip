// Fourier refinement of sampled correlation series on the device,
// Eq. (q-time-pregrid): each series q[0..n-1] (spacing h) is extended by its
// reversed copy to a continuous period of L = 2n samples, its spectrum is
// zero-padded by r (the Nyquist bin split in halves between +L/2 and -L/2)
// and transformed back, giving (n-1) r + 1 samples at spacing h / r that
// reproduce the nodes.
//
// That chain is linear with real coefficients, so the refined series is one
// dense contraction shared by every series:
//   fine[j] = sum_{i<n} T(j, i) q[i],
//   T(j, i) = D(j/r - i) + D(j/r - (2n-1-i)),
//   D(u)    = (1/L) sum over the padded spectrum of e^{2 pi i k u / L}
//           = sin(pi u) cot(pi u / L) / L     (the Nyquist half-bins add cos(pi u)),
// D(0) = 1 and D = 0 at the other integers.  With j = a r + b (phase b), the
// kernel depends on (a - i) and (a + i + 1 - 2n) only, so one table per
// phase, g_b(m) = D(m + b / r) for m in [-(2n-1), n-1], serves every entry.
// Its values are exact to rounding: sin(pi (m + b/r)) = (-1)^m sin(pi b / r)
// and the argument of cot is the rational (m r + b) / (2 n r), reduced in
// integers before the division.
//
// The operator mirrors: T(J, n-1-i) = T(j, i) for J = (n-1) r - j.  So the sum
// and the difference of x[j] and x[J] are contractions of the halves
//   e_i = (q_i + q_{n-1-i}) / 2,  o_i = (q_i - q_{n-1-i}) / 2,  i < ceil(n/2)
// (e of an odd n's middle sample is q/2) with T(j, i) +- T(j, n-1-i): half
// the multiply-adds, for the phases b <= r/2 alone.  Phase 0 is a copy.
//
// The contraction [2 S real columns x n/2] [n/2 x refined samples] runs on the
// FP64 matrix cores (16 x 16 x 4 tiles; their rate is the vector unit's, but
// an operand feeds 16 results instead of one, which takes the loads off the
// critical path).  A wavefront holds one 16 x 16 tile of columns and samples a
// of one phase; the four wavefronts of a block are four phases, which read the
// same e and o and fill the same cache lines of the output.  The operator's
// entries come from the phase's table through LDS: per chunk of i, the sums
// and differences of the table at a - i and a - i - n, and at a + i + 1 - 2n
// and a + i + 1 - n, each a window of chunk + 15 values.  Measured on the
// headline table set (63 series of 820, r = 8): 34 us, 42 us a call with its
// two set-up kernels; a lane per refined sample and four series, with the
// native samples through the scalar path, took 220 and 225 us.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/rift_ile.h"

namespace {

constexpr int PG_IC = 128;    // i per staged chunk
constexpr int PG_STEPS = 8;   // steps of four i whose operands are loaded together
constexpr int PG_PHASES = 4;  // phases (wavefronts) per block
constexpr int PG_LANES = 64;  // refined samples per block, and
constexpr int PG_S = 4;       // series, of the form for short series

// g[b][m + 2n - 1] = D(m + b / r), b < r, m in [-(2n-1), n-1].
__global__ void k_pregrid_table(int n, int r, double* __restrict__ g) {
  const int W = 3 * n - 1;
  const int64_t total = (int64_t)r * W;
  const int64_t Q = 2 * (int64_t)n * r;  // the period in units of 1/r samples
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / W);
    const int m = (int)(e - (int64_t)b * W) - (2 * n - 1);
    double v;
    if (b == 0) {
      v = (m == 0) ? 1.0 : 0.0;  // the nodes (m = -2n, the next multiple of L, is outside the range)
    } else {
      // u / L = p / Q with p = m r + b, reduced to (-Q, Q]
      int64_t p = (int64_t)m * r + b;
      p %= 2 * Q;
      if (p > Q) p -= 2 * Q;
      if (p <= -Q) p += 2 * Q;
      const double x = (double)p / (double)Q;
      const double sgn = (m & 1) ? -1.0 : 1.0;
      v = sgn * sinpi((double)b / (double)r) * cospi(x) / (sinpi(x) * (double)(2 * n));
    }
    g[e] = v;
  }
}

// The halves eo[0][i][c] = e, eo[1][i][c] = o for i < HP (zero past
// ceil(n/2)) and real column c = 2 s + part < CP (zero past 2 S), and the
// nodes fine[s][a r] = q[s][a].
__global__ void k_pregrid_halves(const double* __restrict__ q, int64_t S, int n, int r, int HP, int64_t CP,
                                 double* __restrict__ eo, double* __restrict__ fine) {
  const int64_t Nf = (int64_t)(n - 1) * r + 1;
  const int H = (n + 1) / 2;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t x = t0; x < (int64_t)HP * CP; x += stride) {
    const int i = (int)(x / CP);
    const int64_t c = x - (int64_t)i * CP;
    double e = 0.0, o = 0.0;
    if (i < H && c < 2 * S) {
      const double* qs = q + 2 * (c >> 1) * n + (c & 1);
      const double a = 0.5 * qs[2 * (int64_t)i], b = 0.5 * qs[2 * (int64_t)(n - 1 - i)];
      e = 2 * i == n - 1 ? a : a + b;
      o = a - b;
    }
    eo[x] = e;
    eo[(int64_t)HP * CP + x] = o;
  }
  for (int64_t x = t0; x < S * n; x += stride) {
    const int64_t s = x / n, a = x - (x / n) * n;
    const double2 v = make_double2(q[2 * x], q[2 * x + 1]);
    fine[2 * (s * Nf + a * r)] = v.x;
    fine[2 * (s * Nf + a * r) + 1] = v.y;
  }
}

__global__ void __launch_bounds__(64 * PG_PHASES) k_pregrid(const double* __restrict__ eo, int64_t S, int n, int r,
                                                            int HP, int64_t CP, const double* __restrict__ g,
                                                            double* __restrict__ fine) {
  typedef double D4 __attribute__((ext_vector_type(4)));
  constexpr int LEN = PG_IC + 16;
  __shared__ double win[PG_PHASES][4][LEN];
  const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4, wave = threadIdx.x >> 6;
  const int b = 1 + (int)blockIdx.z * PG_PHASES + wave;
  const int a0 = (int)blockIdx.x * 16;
  const int64_t c0 = (int64_t)blockIdx.y * 16;
  // samples a r + b with a <= n - 2; of the middle phase (its own mirror) the
  // first half.  A wavefront with none still meets the block's barriers.
  const int top = 2 * b == r ? (n - 2) / 2 : n - 2;
  const bool on = 2 * b <= r && a0 <= top;
  const int W = 3 * n - 1;
  const double* gb = g + (int64_t)(on ? b : 0) * W + (2 * n - 1);
  auto G = [&](int m) {  // clamped: entries beyond the table meet zeros of e and o, or samples that are dropped
    return gb[m < -(2 * n - 1) ? -(2 * n - 1) : (m > n - 1 ? n - 1 : m)];
  };
  const double* ec = eo + c0 + col;
  const double* oc = ec + (int64_t)HP * CP;
  D4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
  double ea[PG_STEPS], oa[PG_STEPS], en[PG_STEPS], on_[PG_STEPS];
  auto load = [&](int i, double* e, double* o) {
#pragma unroll
    for (int u = 0; u < PG_STEPS; ++u) {
      const int64_t at = (int64_t)(i + 4 * u + quad) * CP;
      e[u] = ec[at];
      o[u] = oc[at];
    }
  };
  load(0, ea, oa);
  for (int i0 = 0; i0 < HP; i0 += PG_IC) {
    __syncthreads();
    for (int x = lane; x < LEN; x += 64) {
      // win[.][0, 1][x]: a - i = a0 - (i0 + PG_IC - 1) + x;  win[.][2, 3][x]: a + i = a0 + i0 + x
      const int dm = a0 - (i0 + PG_IC - 1) + x, dp = a0 + i0 + x;
      const double w1 = G(dm), w4 = G(dm - n), w2 = G(dp + 1 - 2 * n), w3 = G(dp + 1 - n);
      win[wave][0][x] = w1 + w4;
      win[wave][1][x] = w1 - w4;
      win[wave][2][x] = w2 + w3;
      win[wave][3][x] = w2 - w3;
    }
    __syncthreads();
    const double* m0 = &win[wave][0][col + PG_IC - 1 - quad];
    const double* p0 = &win[wave][2][col + quad];
#pragma unroll
    for (int j = 0; j < PG_IC; j += 4 * PG_STEPS) {
      const int next = i0 + j + 4 * PG_STEPS;
      load(next < HP ? next : 0, en, on_);
#pragma unroll
      for (int u = 0; u < PG_STEPS; ++u) {
        const int d = j + 4 * u;
        const double te = m0[-d] + p0[d], to = m0[LEN - d] + p0[LEN + d];
        E = __builtin_amdgcn_mfma_f64_16x16x4f64(ea[u], te, E, 0, 0, 0);
        O = __builtin_amdgcn_mfma_f64_16x16x4f64(oa[u], to, O, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < PG_STEPS; ++u) {
        ea[u] = en[u];
        oa[u] = on_[u];
      }
    }
  }
  // lane: columns c0 + 4 t + quad, sample (a0 + col) r + b and its mirror
  const int a = a0 + col;
  if (!on || a > top) return;
  const int64_t Nf = (int64_t)(n - 1) * r + 1, j = (int64_t)a * r + b;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t c = c0 + 4 * t + quad;
    if (c >= 2 * S) continue;
    double* o = fine + 2 * (c >> 1) * Nf + (c & 1);
    o[2 * j] = E[t] + O[t];
    o[2 * (Nf - 1 - j)] = E[t] - O[t];
  }
}

// The form for short series: a lane per refined sample and four series, the series'
// native samples uniform across the block (scalar loads), two table reads per tap.
// Native times are copied, as in the matrix form: a sample that is not finite then
// stays out of the others' native times.
__global__ void __launch_bounds__(PG_LANES) k_pregrid_lanes(const double* __restrict__ q, int64_t S, int n,
                                                            int r, const double* __restrict__ g,
                                                            double* __restrict__ fine) {
  const int64_t Nf = (int64_t)(n - 1) * r + 1;
  const int64_t j0 = (int64_t)blockIdx.x * PG_LANES + threadIdx.x;
  const bool live = j0 < Nf;
  const int64_t j = live ? j0 : Nf - 1;
  const int a = (int)(j / r), b = (int)(j - (int64_t)(j / r) * r);
  const int W = 3 * n - 1;
  const double* gb = g + (int64_t)b * W + (2 * n - 1);  // gb[m], m in [-(2n-1), n-1]
  const int64_t s0 = (int64_t)blockIdx.y * PG_S;
  const int ns = (int)std::min<int64_t>(PG_S, S - s0);
  double acc[2 * PG_S];
#pragma unroll
  for (int c = 0; c < 2 * PG_S; ++c) acc[c] = 0.0;
  const double* qs = q + 2 * s0 * (int64_t)n;
  int i = 0;
  for (; i + 4 <= n; i += 4) {
    double t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = gb[a - (i + u)] + gb[a + (i + u) + 1 - 2 * n];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < PG_S; ++c) {
        if (c < ns) {
          acc[2 * c] = fma(t[u], qs[2 * ((int64_t)c * n + i + u)], acc[2 * c]);
          acc[2 * c + 1] = fma(t[u], qs[2 * ((int64_t)c * n + i + u) + 1], acc[2 * c + 1]);
        }
      }
  }
  for (; i < n; ++i) {
    const double t = gb[a - i] + gb[a + i + 1 - 2 * n];
#pragma unroll
    for (int c = 0; c < PG_S; ++c) {
      if (c < ns) {
        acc[2 * c] = fma(t, qs[2 * ((int64_t)c * n + i)], acc[2 * c]);
        acc[2 * c + 1] = fma(t, qs[2 * ((int64_t)c * n + i) + 1], acc[2 * c + 1]);
      }
    }
  }
  if (!live) return;
#pragma unroll
  for (int c = 0; c < PG_S; ++c) {
    if (c < ns) {
      double* o = fine + 2 * ((s0 + c) * Nf + j);
      const double* node = qs + 2 * ((int64_t)c * n + a);
      o[0] = b ? acc[2 * c] : node[0];
      o[1] = b ? acc[2 * c + 1] : node[1];
    }
  }
}

// The matrix form pads the halves to 128 and a tile to 16 samples, and takes two
// set-up launches; a lane per sample has neither.  Measured (us, lanes against
// matrix): 2e5 series of 8, r = 4 84, 741; of 24, r = 2 153, 1111; 2e4 of 32, r = 2 38,
// 106; 2e5 of 48, r = 3 948, 1719; 16 of 64, r = 8 29, 42; 1000 of 96, r = 4 34, 43; but
// 2e4 of 64, r = 4 323, 212; 1000 of 96, r = 16 76, 42; 2e5 of 48 copied (r = 1) 503,
// 386; 168 of 128, r = 8 42, 35.
bool pregrid_by_lanes(int64_t S, int n, int r) {
  return n <= 32 || (n <= 48 && r > 1) || (n <= 96 && (double)S * n * n * r <= 5.0e7);
}

}  // namespace

extern "C" int rift_ile_pregrid(const double* q, int64_t n_series, int32_t n, int32_t r, double* fine, void* stream) {
  if (n_series < 0 || n < 2 || r < 1 || r > 64) return RIFT_EINVAL;
  if ((int64_t)(n - 1) * r + 1 > ((int64_t)1 << 28) || n > (1 << 24)) return RIFT_EINVAL;
  if (n_series == 0) return RIFT_OK;
  if (!q || !fine || (((uintptr_t)q) & 7u) || (((uintptr_t)fine) & 7u)) return RIFT_EINVAL;
  if ((n_series + 3) / 4 > 65535) return RIFT_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  const int64_t tab = (int64_t)r * (3 * n - 1);
  const bool lanes = pregrid_by_lanes(n_series, n, r);
  const int HP = ((n + 1) / 2 + PG_IC - 1) / PG_IC * PG_IC;
  const int64_t CP = (2 * n_series + 15) / 16 * 16;
  double* g = nullptr;
  if (hipMallocAsync((void**)&g, sizeof(double) * (tab + (lanes ? 0 : 2 * HP * CP)), st) != hipSuccess) {
    (void)hipGetLastError();
    return RIFT_ENOMEM;
  }
  hipLaunchKernelGGL(k_pregrid_table, dim3((unsigned)std::min<int64_t>((tab + 255) / 256, 4096)), dim3(256), 0, st, n,
                     r, g);
  if (lanes) {
    const int64_t Nf = (int64_t)(n - 1) * r + 1;
    hipLaunchKernelGGL(k_pregrid_lanes, dim3((unsigned)((Nf + PG_LANES - 1) / PG_LANES), (unsigned)((n_series + PG_S - 1) / PG_S)),
                       dim3(PG_LANES), 0, st, q, n_series, (int)n, (int)r, (const double*)g, fine);
  } else {
    double* eo = g + tab;
    hipLaunchKernelGGL(k_pregrid_halves, dim3((unsigned)std::min<int64_t>((HP * CP + 255) / 256, 4096)), dim3(256), 0,
                       st, q, n_series, (int)n, (int)r, HP, CP, eo, fine);
    const int phases = r / 2;  // 1 .. r / 2
    if (phases > 0)
      hipLaunchKernelGGL(k_pregrid,
                         dim3((unsigned)((n - 1 + 15) / 16), (unsigned)(CP / 16), (unsigned)((phases + PG_PHASES - 1) / PG_PHASES)),
                         dim3(64 * PG_PHASES), 0, st, (const double*)eo, n_series, (int)n, (int)r, HP, CP,
                         (const double*)g, fine);
  }
  int rc = hipGetLastError() == hipSuccess ? RIFT_OK : RIFT_EDEVICE;
  if (hipFreeAsync(g, st) != hipSuccess && !rc) rc = RIFT_EDEVICE;
  return rc;
}
