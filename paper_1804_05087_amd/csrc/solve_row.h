// Row scans of the per-mode Chebyshev-tau solve and its adjoint (solve_reg.h).
//
// Every sequential piece of the solve is a first-order linear recurrence along
// one parity chain n = p, p+2, ..., (chain position k, n = p + 2k):
//   quasi-tridiagonal back substitution  p_k = a_k + b_k p_{k+1}
//   forward pass                          P_k = p_k + q_k P_{k-1}
//   Chebyshev derivative                  D_k = c_k + D_{k+1}
// and the same shapes in the transposed (adjoint) sweeps. x_k = a_k + b_k x_{k-1}
// is the composition of the affine maps f_k(x) = a_k + b_k x, which is
// associative, so one 16-lane row of the wave evaluates a chain as a segmented
// scan: each lane composes the E consecutive maps it owns (k = l E + e, l = lane
// within the row), a Hillis-Steele scan over the row combines them, and each
// lane replays its own maps. The scan steps move data with DPP row shifts
// (row_shr / row_shl: from the lane d below / above within the row; lanes whose
// source lies outside the row receive the identity map), so a chain never
// leaves the vector registers. The four rows of a wave run four chains in one
// instruction stream.
#pragma once

#include <hip/hip_runtime.h>

#include "solve_core.h"

namespace sp {

struct Aff {
  cd a;
  double b;
};

// apply `earlier`, then `later`
__device__ inline Aff aff_compose(Aff earlier, Aff later) {
  return {later.a + earlier.a * later.b, later.b * earlier.b};
}

constexpr int kDppRowShl = 0x100;  // lane l <- lane l + n (same row)
constexpr int kDppRowShr = 0x110;  // lane l <- lane l - n (same row)
constexpr int kDppRowRor = 0x120;  // lane l <- lane (l - n) mod 16

// One DPP move of a double; lanes without a source in the row keep `old`.
template <int CTRL>
__device__ inline double dpp_mov(double v, double old) {
  const long long vi = __double_as_longlong(v);
  const long long oi = __double_as_longlong(old);
  const int lo = __builtin_amdgcn_update_dpp((int)oi, (int)vi, CTRL, 0xF, 0xF, false);
  const int hi =
      __builtin_amdgcn_update_dpp((int)(oi >> 32), (int)(vi >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

template <int CTRL>
__device__ inline Aff aff_dpp(Aff m) {
  return {cd(dpp_mov<CTRL>(m.a.re, 0.0), dpp_mov<CTRL>(m.a.im, 0.0)), dpp_mov<CTRL>(m.b, 1.0)};
}

template <int CTRL>
__device__ inline cd cd_dpp(cd v) {
  return cd(dpp_mov<CTRL>(v.re, 0.0), dpp_mov<CTRL>(v.im, 0.0));
}

// Sum over the 16 lanes of the row, returned in every lane of the row.
__device__ inline cd row_sum(cd v) {
  v = v + cd_dpp<kDppRowRor | 8>(v);
  v = v + cd_dpp<kDppRowRor | 4>(v);
  v = v + cd_dpp<kDppRowRor | 2>(v);
  v = v + cd_dpp<kDppRowRor | 1>(v);
  return v;
}

// x_k = a_k + b_k x_{k-1} for k = 0 .. 16E-1 (x_{-1} = x_init), blocked layout.
template <int E>
__device__ inline void rec_up(const cd (&a)[E], const double (&b)[E], cd x_init, cd (&x)[E]) {
  Aff m{a[0], b[0]};
#pragma unroll
  for (int e = 1; e < E; ++e) m = aff_compose(m, Aff{a[e], b[e]});
  m = aff_compose(aff_dpp<kDppRowShr | 1>(m), m);
  m = aff_compose(aff_dpp<kDppRowShr | 2>(m), m);
  m = aff_compose(aff_dpp<kDppRowShr | 4>(m), m);
  m = aff_compose(aff_dpp<kDppRowShr | 8>(m), m);
  const Aff ex = aff_dpp<kDppRowShr | 1>(m);  // maps of all lower lanes (identity in lane 0)
  cd xv = ex.a + x_init * ex.b;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    xv = a[e] + xv * b[e];
    x[e] = xv;
  }
}

// x_k = a_k + b_k x_{k+1} for k = 16E-1 .. 0 (x_{16E} = x_init), blocked layout.
template <int E>
__device__ inline void rec_down(const cd (&a)[E], const double (&b)[E], cd x_init, cd (&x)[E]) {
  Aff m{a[E - 1], b[E - 1]};
#pragma unroll
  for (int e = E - 2; e >= 0; --e) m = aff_compose(m, Aff{a[e], b[e]});
  m = aff_compose(aff_dpp<kDppRowShl | 1>(m), m);
  m = aff_compose(aff_dpp<kDppRowShl | 2>(m), m);
  m = aff_compose(aff_dpp<kDppRowShl | 4>(m), m);
  m = aff_compose(aff_dpp<kDppRowShl | 8>(m), m);
  const Aff ex = aff_dpp<kDppRowShl | 1>(m);  // maps of all higher lanes (identity in lane 15)
  cd xv = ex.a + x_init * ex.b;
#pragma unroll
  for (int e = E - 1; e >= 0; --e) {
    xv = a[e] + xv * b[e];
    x[e] = xv;
  }
}

// Element loads use indexes clamped into the chain and 0/1 masks applied to the
// loaded values instead of per-element branches: a load under a per-lane
// condition is compiled into its own branch followed by a wait for it, which
// serialises the LDS round trips.
__device__ inline double mask(bool c) { return c ? 1.0 : 0.0; }

}  // namespace sp
