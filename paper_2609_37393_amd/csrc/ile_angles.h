// The polarisation and phase rules on a sample's angular coefficients, after
// the likelihood kernel's data passes (angles.hip).
#pragma once

#include "ile_device.h"

namespace rift {

// The rule over polarisation (Sec. "Angles: finite harmonic content"): with psi
// uniform on [0, pi), L_psi = (1 / 2 pi) int_0^{2 pi} e^{q(u)} du by
//   0: the periodic trapezoid rule on n points (the product grid),
//   1: Laplace's method at the dominant maximum u* (Eq. (ap:psilaplace)),
//      L_psi = e^{q(u*)} sqrt(2 pi / A) / (2 pi), A = -q''(u*), where A >= 100
//      (relative error O(1/A) below ~1e-3); a q without such a maximum (weak
//      signal, or two peaks merging) takes the trapezoid rule on 256 points,
//   2: the cells between the stationary points (Eq. (ap:psicells)).
struct PsiRule {
  int32_t method;
  int32_t n;
};

// Doubles of the uniform tables a rule needs.
size_t psi_tables_len(const PsiRule& r);
size_t erai_tables_len(int n_phi, int n_psi, int m_max);

// The values of a piece's samples: sample i's is at L[i], or, in a binned batch
// (rec set: the piece's records of eight doubles, the sample's index in the last
// one's upper 48 bits), at L[index].
struct PsiOut {
  double* L;
  const double* rec;
  __device__ __forceinline__ int64_t at(int64_t i) const {
    return rec ? (int64_t)__double_as_longlong(as_global(rec)[8 * i + 7]) >> 16 : i;
  }
};

// coef [PSI_ROWS][stride] of samples 0 .. cnt-1, tab the workspace of the
// tables; the values are NaN (poisoned) or 0 on entry and ln L_psi on return.
int psi_tables(const PsiRule& r, double* tab, hipStream_t st);
int run_psi(const PsiRule& r, int64_t cnt, const double* coef, int64_t stride, const double* tab, const PsiOut& out,
            hipStream_t st);
// ang [2 nd + 3 nq][stride]; the n_phi x n_psi grid.
int erai_tables(int n_phi, int n_psi, int m_max, double* tab, hipStream_t st);
int run_erai(int64_t cnt, int n_phi, int n_psi, int m_max, const double* ang, int64_t stride, const double* tab,
             const PsiOut& out, hipStream_t st);

}  // namespace rift
