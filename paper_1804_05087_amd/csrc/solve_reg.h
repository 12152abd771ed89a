// Register-resident building blocks of the per-mode Chebyshev-tau solve and its adjoint.
//
// A parity chain of coefficients lives in the vector registers of one 16-lane
// row: lane l of the row holds the E consecutive chain positions k = l E + e,
// position k being the coefficient n = n0 + 2 k. Every step of the solve maps
// such registers to such registers: the stencils of the quasi-tridiagonal form
// need positions k - 1 and k + 1 (a DPP shift by one lane for the outermost
// element), the recurrences are row scans, the sums row reductions. So the
// steps follow one another without a trip through LDS.
//
// Rows 0, 1 of a wave carry the class of v parity pv = row: v on the chain
// n0 = pv and P (and u_par, div F) on n0 = pv - 1, of the other parity. With
// these two origins D maps position k of v to position k of P's chain, and
// position k + 1 of P to position k of v's, for either class, so both rows run
// the same instructions. (For pv = 0 position 0 of P's chain would be
// n = -1: it holds a value nobody uses, since every weight there is zero.)
// The weights (hwp) are zero for n < 2 and n > N, which ends every recurrence
// at the ends of its chain without masks; entries past a chain's end only ever
// meet zero weights, so they need to be finite, not zero.
//
// What bounds it: one mode is one chain of dependent steps. With every step's
// operands in LDS arrays indexed by n (ten arrays, three to four LDS round trips
// a step) the solve took 6.3 / 8.5 / 13.8 / 95.8 us at 16x17x16, 32x33x32,
// 48x65x48 and 96x97x96; with the steps in registers it takes 6.1 / 7.6 / 11.9 /
// 55.2 us: a sweep fell from 2.8 k to 1.7 k cycles, and at ny = 97 the seven LDS
// arrays no longer needed (11 KB a mode) let more modes share a CU. The adjoint solve's
// steps are these transposed, in reverse order.
#pragma once

#include <hip/hip_runtime.h>

#include "solve_core.h"
#include "solve_row.h"

namespace sp {

// Row length of the zero-padded weight table [3][hwp_row]: entry n at n + 1,
// n = -1 .. N + 1.
__host__ __device__ constexpr int hwp_row(int ny) { return ny + 2; }

// Elements per lane so that both chains of a class (the even-n one from
// n = 0, or the odd-n one from n = -1, up to N) fit 16 lanes.
__host__ __device__ constexpr int solve_reg_elems(int ny) { return (ny / 2 + 16) / 16; }

// Factors of one operator (D^2 - lam) on one chain, at this lane's positions,
// from the record and the weights in LDS.
template <int E>
struct RegSweep {
  double w1[E], w2[E], w3[E], id[E], Q[E];
  double inv_sum, lam;
  // rec: the operator's block of the mode record (inv_den, Q, inv_sum)
  __device__ RegSweep(const double* hwp, const double* rec, int N, int n0, double lam_, int l)
      : inv_sum(rec[2 * (N + 1) + (n0 & 1)]), lam(lam_) {
    const int n1 = N + 1;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = n0 + 2 * (l * E + e);
      const int nw = n <= N ? n + 1 : N + 2;
      w1[e] = hwp[nw];
      w2[e] = hwp[hwp_row(n1) + nw];
      w3[e] = hwp[2 * hwp_row(n1) + nw];
      const int nc = n < 0 ? 0 : (n > N ? N : n);
      id[e] = rec[nc];
      Q[e] = rec[n1 + nc];
    }
  }
};

// Chosen by value (a conditional between two array elements would be one between
// their addresses, which keeps the arrays out of registers).
__device__ inline cd pick(bool c, cd a, cd b) { return cd(c ? a.re : b.re, c ? a.im : b.im); }

// s_k = sum of c over the positions k' >= k of the row.
template <int E>
__device__ inline void suffix_sum(const cd (&c)[E], cd (&s)[E]) {
  cd t = c[E - 1];
#pragma unroll
  for (int e = E - 2; e >= 0; --e) t = t + c[e];
  t = t + cd_dpp<kDppRowShl | 1>(t);
  t = t + cd_dpp<kDppRowShl | 2>(t);
  t = t + cd_dpp<kDppRowShl | 4>(t);
  t = t + cd_dpp<kDppRowShl | 8>(t);
  cd x = cd_dpp<kDppRowShl | 1>(t);  // of all higher lanes (zero in lane 15)
#pragma unroll
  for (int e = E - 1; e >= 0; --e) {
    x = c[e] + x;
    s[e] = x;
  }
}

// s_k = sum of c over the positions k' <= k of the row.
template <int E>
__device__ inline void prefix_sum(const cd (&c)[E], cd (&s)[E]) {
  cd t = c[0];
#pragma unroll
  for (int e = 1; e < E; ++e) t = t + c[e];
  t = t + cd_dpp<kDppRowShr | 1>(t);
  t = t + cd_dpp<kDppRowShr | 2>(t);
  t = t + cd_dpp<kDppRowShr | 4>(t);
  t = t + cd_dpp<kDppRowShr | 8>(t);
  cd x = cd_dpp<kDppRowShr | 1>(t);  // of all lower lanes (zero in lane 0)
#pragma unroll
  for (int e = 0; e < E; ++e) {
    x = c[e] + x;
    s[e] = x;
  }
}

// g with (D^2 - lam) g = r on the chain (rows 0..N-2) and sum g_n = beta:
// sweep_solve's two recurrences (solve_core.h) on registers.
template <int E>
__device__ inline void rsweep(const RegSweep<E>& f, const cd (&r)[E], cd beta, cd (&g)[E]) {
  cd a[E], x[E];
  double b[E];
  const cd lower = cd_dpp<kDppRowShr | 1>(r[E - 1]);  // position l E - 1
  const cd upper = cd_dpp<kDppRowShl | 1>(r[0]);      // position (l + 1) E
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const cd rm = pick(e == 0, lower, r[e > 0 ? e - 1 : 0]);
    const cd rp = pick(e == E - 1, upper, r[e < E - 1 ? e + 1 : 0]);
    a[e] = (rm * f.w1[e] + r[e] * f.w2[e] + rp * f.w3[e]) * f.id[e];
    b[e] = f.lam * f.w3[e] * f.id[e];  // -cc / den
  }
  rec_down<E>(a, b, cd(0.0), x);
#pragma unroll
  for (int e = 0; e < E; ++e) b[e] = f.lam * f.w1[e] * f.id[e];  // q
  rec_up<E>(x, b, cd(0.0), a);
  cd s = a[0];
#pragma unroll
  for (int e = 1; e < E; ++e) s = s + a[e];
  s = row_sum(s);
  const cd g0 = (beta - s) * f.inv_sum;
#pragma unroll
  for (int e = 0; e < E; ++e) g[e] = a[e] + g0 * f.Q[e];  // Q = 1 at the first position
}

// rsweep transposed (beta = 0): r = its adjoint of the right-hand side from the adjoint g
// of the solution, which is zero past the chain.
template <int E>
__device__ inline void rsweep_T(const RegSweep<E>& f, const cd (&g)[E], cd (&r)[E]) {
  cd s = g[0] * f.Q[0];
#pragma unroll
  for (int e = 1; e < E; ++e) s = s + g[e] * f.Q[e];
  s = row_sum(s) * (-f.inv_sum);
  cd a[E], x[E];
  double b[E];
  // the forward pass transposed: x_k = (g_k + s) + q_{k+1} x_{k+1}
  const double qn = dpp_mov<kDppRowShl | 1>(f.lam * f.w1[0] * f.id[0], 0.0);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    a[e] = g[e] + s;
    const int u = e < E - 1 ? e + 1 : 0;
    b[e] = (e == E - 1) ? qn : f.lam * f.w1[u] * f.id[u];
  }
  rec_down<E>(a, b, cd(0.0), x);
  // the back substitution transposed: a_k = x_k + (-cc / den)_{k-1} a_{k-1}
  const double cp = dpp_mov<kDppRowShr | 1>(f.lam * f.w3[E - 1] * f.id[E - 1], 0.0);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int u = e > 0 ? e - 1 : 0;
    b[e] = (e == 0) ? cp : f.lam * f.w3[u] * f.id[u];
  }
  rec_up<E>(x, b, cd(0.0), a);
  // the right-hand side's combination transposed
#pragma unroll
  for (int e = 0; e < E; ++e) a[e] = a[e] * f.id[e];
  const cd up = cd_dpp<kDppRowShl | 1>(a[0] * f.w1[0]);
  const cd dn = cd_dpp<kDppRowShr | 1>(a[E - 1] * f.w3[E - 1]);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int u = e < E - 1 ? e + 1 : 0, v = e > 0 ? e - 1 : 0;
    r[e] = a[e] * f.w2[e] + pick(e == E - 1, up, a[u] * f.w1[u]) +
           pick(e == 0, dn, a[v] * f.w3[v]);
  }
}

}  // namespace sp
