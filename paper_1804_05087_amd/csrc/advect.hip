// The BEFE step with the laminar advection moved into the implicit operator
// (paper Sec. 3.6, the proposed remedy for the Krylov counts at high Re):
//
//   (I - dt (L + M)) Phi~(U) = U + dt (N(U) - M U),
//   M u = -( i k_x y u + v, i k_x y v, i k_x y w )    per Fourier mode,
//
// the linearisation of the advection about U_lam = y e_x in convective form.
// Multiplication by y couples neighbouring Chebyshev coefficients of both
// parities, so the per-mode system no longer splits into the parity chains of
// the Stokes solve. The plan therefore builds, once per (Re, dt), each mode's
// dense solution operator S~_k (the tau system's map from the 3 (N-1) used
// right-hand-side coefficients to the 3 (N+1) velocity coefficients) by LU with
// partial pivoting and iterative refinement with extended-precision residuals,
// and the step applies it as a per-mode matrix-vector product. The mean mode
// (k_x = 0, v = 0) is unchanged: its operator is the Dirichlet Helmholtz solve.
//
// Two symmetries of the advected system quarter what is stored and read:
//  - conjugation with z -> -z (w -> -w): S~(-k_x, k_z) = R conj(S~(k_x, k_z)) R,
//    R = diag(1, 1, -1) over the components, so m_x and -m_x share an operator;
//  - that, with the rotation (x, y) -> (-x, -y) (u, v -> -u, -v, a_n -> (-1)^n a_n),
//    maps a mode to itself and conjugates it: with coefficients scaled by p_n = 1
//    (n even), i (n odd) the operator is real (its entry is the complex one times
//    p_col / p_row, whose imaginary part vanishes).
// So a mode pair's operator is a real 3 (N-1) x 3 (N+1) matrix applied to four
// real vectors, the parts of the two modes' scaled right-hand sides.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <complex>
#include <thread>
#include <type_traits>
#include <vector>

#include "device_common.h"
#include "host_math.h"
#include "solve_core.h"
#include "sp_internal.h"

namespace sp {

namespace {

template <typename TS>
struct OpVec2;
template <>
struct OpVec2<double> {
  typedef double T __attribute__((ext_vector_type(2)));
};
template <>
struct OpVec2<float> {
  typedef float T __attribute__((ext_vector_type(2)));
};

constexpr int kAdvRows = 128;  // row pairs a pass of the block covers
constexpr int kAdvDepth = 8;   // columns in flight per thread

// out_k = S~_k (g_k + xa x_k + i k_x Y x_k + (x_v, 0, 0)) on the used coefficients for
// the modes (m_x, m_z) and (-m_x, m_z) of block m_x nzm + m_z (one mode at m_x = 0);
// the blocks past the pairs write the Nyquist modes' zeros. out may alias x.
// AN = 0: g (canonical) holds the right-hand side with xa x added already.
// AN = 1: g = Tinv nv is formed here, in FP64, from the y-valued product fields
// (folded halves and table as in the Stokes solve's fused analysis).
// Smean: the (0,0) mode's operator, in FP64 for either TS.
// wall: the (0,0) mode's response to the wall velocities, or NULL (homogeneous).
// RES: out = oa (.) + ob x in the Hermitian form (the m_z = 0 plane's -m_x entries
// are conjugates of the m_x ones, the (0,0) mode real); out must not alias x.
//
// Bound by the operators' bytes: 163 MB (FP64) at 48x65x48, read in about 40 us with
// the analysis in front of it; as complex matrices, one per mode, they were 737 MB
// and 130 us. A thread owns two rows (16-byte loads) and half of the columns, eight
// loads ahead of their use; the four vectors' entries come from LDS (broadcast).
template <typename TS, int AN, bool RES>
__global__ void __launch_bounds__(256)
    k_adv_apply(const double2* __restrict__ g, const double2* x, double xa,
                const TS* __restrict__ S, const double* __restrict__ Smean,
                const double* __restrict__ wall, double2* out, int nx,
                int ny, int nzh, double alpha, const double2* __restrict__ nv,
                const double* __restrict__ th, double oa, double ob) {
  extern __shared__ unsigned char smem_raw[];
  const int nzm = nzh - 1, h = nx / 2, N = ny - 1;
  const int nm = N - 1;  // used right-hand-side coefficients of a component
  const int C = 3 * nm, R = 3 * ny, Rp = (R + 1) & ~1;
  const size_t cs = (size_t)nx * nzh * ny;
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= h * nzm) {  // Nyquist: m_x = nx/2 (every m_z), then m_z = nz/2
    const int q = blockIdx.x - h * nzm;
    const int i = q < nzh ? h : q - nzh;
    const int j = q < nzh ? q : nzh - 1;
    const size_t mo = ((size_t)i * nzh + j) * ny;
    for (int t = tid; t < R; t += 256) {
      const int c = t / ny;
      out[c * cs + mo + (t - c * ny)] = make_double2(0.0, 0.0);
    }
    return;
  }
  const int i = blockIdx.x / nzm;
  const int j = blockIdx.x - i * nzm;
  const double kx = alpha * (double)i;
  const bool mean = (i == 0 && j == 0);
  const bool mirror = RES && j == 0 && i > 0;       // -m_x follows from m_x
  const int nmode = (i == 0 || mirror) ? 1 : 2;
  size_t mo[2];
  mo[0] = ((size_t)i * nzh + j) * ny;
  mo[1] = ((size_t)(i == 0 ? 0 : nx - i) * nzh + j) * ny;

  double* vec = reinterpret_cast<double*>(smem_raw);  // [C][4]
  // [6][jh] even and [6][jh] odd halves; afterwards [kAdvRows][8] partial sums
  double2* fold = reinterpret_cast<double2*>(vec + 4 * C);
  const int jh = N / 2 + 1;
  if constexpr (AN == 1) {
    const size_t fs = (size_t)ny * nzm * nx;
    for (int t = tid; t < 3 * nmode * jh; t += 256) {
      const int col = t / jh;  // 3 mode + component
      const int jj = t - col * jh;
      const int md = col / 3;
      const double2* f = nv + (col - 3 * md) * fs + (size_t)j * nx + (md ? nx - i : i);
      const double2 a = f[(size_t)jj * nzm * nx], b = f[(size_t)(N - jj) * nzm * nx];
      const double same = (jj == N - jj) ? 0.0 : 1.0;  // middle point counted once
      fold[col * jh + jj] = make_double2(a.x + same * b.x, a.y + same * b.y);
      fold[(6 + col) * jh + jj] = make_double2((a.x - b.x) * same, (a.y - b.y) * same);
    }
    __syncthreads();
  }
  // the right-hand sides, scaled: entry (component c, coefficient n) of mode md
  for (int t = tid; t < 2 * C; t += 256) {
    const int md = t / C;
    const int e = t - md * C;
    const int c = e / nm;
    const int n = e - c * nm;
    double2 v = make_double2(0.0, 0.0);
    if (md < nmode) {
      const double2* a = x + c * cs + mo[md];
      if constexpr (AN == 1) {
        const double2* f = fold + ((n & 1 ? 6 : 0) + 3 * md + c) * jh;
#pragma unroll 8
        for (int jj = 0; jj < jh; ++jj) {
          const double w = th[(size_t)jj * ny + n];
          v.x += w * f[jj].x;
          v.y += w * f[jj].y;
        }
        v.x += xa * a[n].x;
        v.y += xa * a[n].y;
      } else {
        v = g[c * cs + mo[md] + n];
      }
      if (!mean) {
        double2 y;  // (y a)_n
        if (n == 0) {
          y = make_double2(0.5 * a[1].x, 0.5 * a[1].y);
        } else {
          const double w = (n == 1) ? 1.0 : 0.5;
          y = make_double2(w * a[n - 1].x + 0.5 * a[n + 1].x, w * a[n - 1].y + 0.5 * a[n + 1].y);
        }
        const double k = md ? -kx : kx;
        v.x -= k * y.y;  // + i kx (y a)
        v.y += k * y.x;
        if (c == 0) {
          v.x += x[cs + mo[md] + n].x;  // + v
          v.y += x[cs + mo[md] + n].y;
        }
      }
      // mode m_x: divided by p_n; mode -m_x: R conj(.) R, divided by conj(p_n)
      if (n & 1) v = md ? make_double2(-v.y, v.x) : make_double2(v.y, -v.x);
      if (md && c == 2) v = make_double2(-v.x, -v.y);
    }
    vec[4 * e + 2 * md] = v.x;
    vec[4 * e + 2 * md + 1] = v.y;
  }
  __syncthreads();
  const TS* Sm = S + (size_t)blockIdx.x * C * Rp;
  const int half = tid / kAdvRows;
  const int rt = tid - half * kAdvRows;
  const int c0 = half ? C / 2 : 0;
  const int c1 = half ? C : C / 2;
  double* part = reinterpret_cast<double*>(fold);
  for (int r0 = 0; r0 < Rp / 2; r0 += kAdvRows) {  // uniform
    const int rp = r0 + rt;
    double acc[2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[0][q] = acc[1][q] = 0.0;
    auto columns = [&](auto* M) {
      using V2T = typename OpVec2<typename std::remove_cv<
          typename std::remove_pointer<decltype(M)>::type>::type>::T;
      const V2T* col = reinterpret_cast<const V2T*>(M) + rp;
      const size_t ld = Rp / 2;
      V2T s[kAdvDepth];
#pragma unroll
      for (int q = 0; q < kAdvDepth; ++q) s[q] = col[min(c0 + q, C - 1) * ld];
      for (int cb = c0; cb < c1; cb += kAdvDepth) {
#pragma unroll
        for (int q = 0; q < kAdvDepth; ++q) {
          const V2T w = s[q];
          s[q] = col[min(cb + kAdvDepth + q, C - 1) * ld];  // past the end: re-reads
          if (cb + q < c1) {                                // uniform
            const double* b = vec + 4 * (cb + q);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              acc[0][k] += (double)w.x * b[k];
              acc[1][k] += (double)w.y * b[k];
            }
          }
        }
      }
    };
    if (rp < Rp / 2) {
      if (sizeof(TS) < sizeof(double) && mean)
        columns(Smean);
      else
        columns(Sm);
    }
    __syncthreads();  // the folded columns (first pass) and the last pass' sums are read
    if (half) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        part[k * kAdvRows + rt] = acc[0][k];
        part[(4 + k) * kAdvRows + rt] = acc[1][k];
      }
    }
    __syncthreads();
    if (!half && rp < Rp / 2) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = 2 * rp + q;
        if (r < R) {
          double s[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) s[k] = acc[q][k] + part[(4 * q + k) * kAdvRows + rt];
          const int c = r / ny;
          const int n = r - c * ny;
          for (int md = 0; md < nmode; ++md) {
            const double re = md ? s[2] : s[0], im = md ? s[3] : s[1];
            double2 o = make_double2(re, im);
            if (n & 1) o = md ? make_double2(im, -re) : make_double2(-im, re);
            if (md && c == 2) o = make_double2(-o.x, -o.y);
            if (mean && c == 0 && wall != nullptr) o.x += wall[n];
            if constexpr (RES) {
              const double2 xv = x[c * cs + mo[md] + n];
              o = make_double2(oa * o.x + ob * xv.x, oa * o.y + ob * xv.y);
              if (mean) o.y = 0.0;
              if (mirror) out[c * cs + mo[1] + n] = make_double2(o.x, -o.y);
            }
            out[c * cs + mo[md] + n] = o;
          }
        }
      }
    }
  }
}

}  // namespace

// Operators of the mode pairs: m_x < nx/2, m_z < nz/2, column-major with an even
// column length.
static size_t adv_count(const sp_plan* p) {
  const Dims& d = p->d;
  return (size_t)(d.nx / 2) * d.nzm * 3 * (d.N - 1) * ((3 * d.ny + 1) & ~1);
}

// Entry of the real operator from entry z of the complex one: z p_col / p_row, p = 1
// (n even), i (n odd).
__host__ __device__ static inline double adv_real_entry(double re, double im, int row_n, int col_n) {
  if (((row_n ^ col_n) & 1) == 0) return re;
  return (col_n & 1) ? -im : im;
}

namespace {

// ---- The operators built on the device, one workgroup per mode pair ----

__device__ inline double d1_coef(int n, int m) {  // (D)_{nm}: d/dy on coefficients
  return (m > n && ((m + n) & 1)) ? (n == 0 ? 1.0 : 2.0) * m : 0.0;
}
__device__ inline double d2_coef(int n, int m) {  // (D D)_{nm} = m (m^2 - n^2) / c_n
  return (m >= n + 2 && ((m + n) & 1) == 0)
             ? (double)m * ((double)m * m - (double)n * n) / (n == 0 ? 2.0 : 1.0)
             : 0.0;
}

// Entry (r, c) of the tau matrix that adv_mode_matrix assembles.
__device__ double2 adv_entry(int N, double kx, double kz, double re, double diag, int r, int c) {
  const int n1 = N + 1, V = n1, W = 2 * n1, P = 3 * n1, nm = 3 * (N - 1);
  double er = 0.0, ei = 0.0;
  if (r < nm) {  // momentum component comp on T_n
    const int comp = r / (N - 1), n = r - comp * (N - 1), off = comp * n1;
    if (c >= off && c < off + n1) {
      const int m = c - off;
      er = d2_coef(n, m) / re - (m == n ? diag : 0.0);
      double yc = 0.0;  // coefficient of a_m in (y a)_n
      if (n == 0) {
        if (m == 1) yc = 0.5;
      } else {
        if (m == n - 1) yc = (n == 1) ? 1.0 : 0.5;
        if (m == n + 1) yc = 0.5;
      }
      ei = -kx * yc;
    }
    if (comp == 0) {
      if (c == V + n) er -= 1.0;
      if (c == P + n) er = 0.0, ei = -kx;
    } else if (comp == 1) {
      if (c >= P) er = -d1_coef(n, c - P), ei = 0.0;
    } else {
      if (c == P + n) er = 0.0, ei = -kz;
    }
  } else if (r < nm + 6) {  // no-slip rows: u(1) = 0, u(-1) = 0 for u, v, w
    const int q = r - nm, off = (q >> 1) * n1;
    if (c >= off && c < off + n1) er = (q & 1) ? (((c - off) & 1) ? -1.0 : 1.0) : 1.0;
  } else {  // continuity on T_n
    const int n = r - nm - 6;
    if (c == n) ei = kx;
    else if (c >= V && c < V + n1) er = d1_coef(n, c - V);
    else if (c == W + n) ei = kz;
  }
  return make_double2(er, ei);
}

// Double-double accumulator (Knuth's two-sum and the FMA two-product).
struct DD {
  double hi = 0.0, lo = 0.0;
  __device__ void add(double p, double pe) {
    const double s = hi + p;
    const double bb = s - hi;
    lo += ((hi - (s - bb)) + (p - bb)) + pe;
    hi = s;
  }
  __device__ void add_prod(double a, double b) {
    const double p = a * b;
    add(p, fma(a, b, -p));
  }
};

// X_c <- (LU)^{-1} P X_c (X n x C, row-major) with the workgroup's factors
// and pivots; one thread per column, no barriers. The inner products run over
// every entry (zeros included) so that the unrolled loads overlap instead of
// each waiting on a test of the previous one.
__device__ void adv_lu_solve_col(const double2* __restrict__ LU, const int* piv, int n, int C,
                                 double2* __restrict__ X, int c) {
  for (int k = 0; k < n; ++k) {
    const int p = piv[k];
    if (p != k) {
      const double2 t = X[(size_t)k * C + c];
      X[(size_t)k * C + c] = X[(size_t)p * C + c];
      X[(size_t)p * C + c] = t;
    }
  }
  for (int r = 1; r < n; ++r) {
    double sr = X[(size_t)r * C + c].x, si = X[(size_t)r * C + c].y;
    const double2* Lr = LU + (size_t)r * n;
#pragma unroll 8
    for (int q = 0; q < r; ++q) {
      const double2 l = Lr[q];
      const double2 x = X[(size_t)q * C + c];
      sr -= l.x * x.x - l.y * x.y;
      si -= l.x * x.y + l.y * x.x;
    }
    X[(size_t)r * C + c] = make_double2(sr, si);
  }
  for (int r = n - 1; r >= 0; --r) {
    double sr = X[(size_t)r * C + c].x, si = X[(size_t)r * C + c].y;
    const double2* Ur = LU + (size_t)r * n;
#pragma unroll 8
    for (int q = r + 1; q < n; ++q) {
      const double2 u = Ur[q];
      const double2 x = X[(size_t)q * C + c];
      sr -= u.x * x.x - u.y * x.y;
      si -= u.x * x.y + u.y * x.x;
    }
    const double2 d = Ur[r];
    const double den = d.x * d.x + d.y * d.y;
    X[(size_t)r * C + c] = make_double2((sr * d.x + si * d.y) / den, (si * d.x - sr * d.y) / den);
  }
}

// Row r of -e_c - A x_c accumulated in double-double over the non-zero
// entries of row r only, which the tau matrix's structure fixes: in a
// momentum row n of component comp its own block at m = n - 1, n, n + 1 and
// m = n + 2, n + 4, ... (second derivative), the coupling entries (v and p
// for u, the pressure gradient); all of its block in a no-slip row; u, w and
// the odd-offset derivative of v in a continuity row. The entries come from
// adv_entry, so A is never stored.
__device__ double2 adv_residual_row(int N, double kx, double kz, double re, double diag, int r,
                                    const double2* __restrict__ X, int C, int c) {
  const int n1 = N + 1, V = n1, W = 2 * n1, P = 3 * n1, nm = 3 * (N - 1);
  DD sr, si;
  if (r == c) sr.hi = -1.0;
  auto acc = [&](int q) {
    const double2 a = adv_entry(N, kx, kz, re, diag, r, q);
    const double2 x = X[(size_t)q * C + c];
    sr.add_prod(-a.x, x.x);
    sr.add_prod(a.y, x.y);
    si.add_prod(-a.x, x.y);
    si.add_prod(-a.y, x.x);
  };
  if (r < nm) {
    const int comp = r / (N - 1), n = r - comp * (N - 1), off = comp * n1;
    if (n >= 1) acc(off + n - 1);
    acc(off + n);
    acc(off + n + 1);
    for (int m = n + 2; m <= N; m += 2) acc(off + m);
    if (comp == 0) {
      acc(V + n);
      acc(P + n);
    } else if (comp == 1) {
      for (int m = n + 1; m <= N; m += 2) acc(P + m);
    } else {
      acc(P + n);
    }
  } else if (r < nm + 6) {
    const int off = ((r - nm) >> 1) * n1;
    for (int m = 0; m <= N; ++m) acc(off + m);
  } else {
    const int n = r - nm - 6;
    acc(n);
    for (int m = n + 1; m <= N; m += 2) acc(V + m);
    acc(W + n);
  }
  return make_double2(sr.hi + sr.lo, si.hi + si.lo);
}

// Column c of the operator: solve A x = -e_c with the workgroup's factors,
// refine twice with residuals accumulated in double-double, and write the
// first R rows of x, as real entries, to column c of the mode's operator Sm
// (column length Rp).
__device__ void adv_solve_refine(const double2* __restrict__ LU, const int* piv, int N, double kx,
                                 double kz, double re, double diag, int C, int R,
                                 double2* __restrict__ X, double2* __restrict__ Rw, int c,
                                 int Rp, double* __restrict__ Sm) {
  const int n4 = 4 * (N + 1);
  for (int r = 0; r < n4; ++r) X[(size_t)r * C + c] = make_double2(r == c ? -1.0 : 0.0, 0.0);
  adv_lu_solve_col(LU, piv, n4, C, X, c);
  for (int it = 0; it < 2; ++it) {
    for (int r = 0; r < n4; ++r)
      Rw[(size_t)r * C + c] = adv_residual_row(N, kx, kz, re, diag, r, X, C, c);
    adv_lu_solve_col(LU, piv, n4, C, Rw, c);
    for (int r = 0; r < n4; ++r) {
      const double2 x = X[(size_t)r * C + c], d = Rw[(size_t)r * C + c];
      X[(size_t)r * C + c] = make_double2(x.x + d.x, x.y + d.y);
    }
  }
  const int cn = c % (N - 1);
  for (int r = 0; r < R; ++r) {
    const double2 z = X[(size_t)r * C + c];
    Sm[(size_t)c * Rp + r] = adv_real_entry(z.x, z.y, r % (N + 1), cn);
  }
}

constexpr int kAdvMaxN4 = 4 * 130;  // ny <= 129

// One workgroup per mode of modes[]: assemble the tau matrix A, LU with
// partial pivoting (the first row of largest modulus, as on the host; only
// the rows with a non-zero multiplier are updated), solve A X = -E for the 3 (N-1) used
// right-hand sides (columns strided over the threads), refine twice with residuals
// accumulated in double-double, and write the first 3 (N+1) rows of X as the
// mode's operator in the layout of k_adv_apply. ws holds, per workgroup,
// LU (n4 x n4) and X and the residual (n4 x C). status[b] = 1 if the
// system is singular.
__global__ void __launch_bounds__(256)
    k_adv_build(const int* __restrict__ modes, int N, int nx, int nzh, double alpha, double gamma,
                double re, double inv_dt, double2* __restrict__ ws, size_t ws_stride,
                double* __restrict__ S, int* __restrict__ status) {
  __shared__ int piv[kAdvMaxN4];
  __shared__ int rows[kAdvMaxN4];
  __shared__ double bval[256];
  __shared__ int bidx[256];
  __shared__ int nrows;
  const int tid = threadIdx.x;
  const int n1 = N + 1, n4 = 4 * n1, C = 3 * (N - 1), R = 3 * n1, Rp = (R + 1) & ~1;
  const int mode = modes[blockIdx.x];
  const int i = mode / nzh, j = mode - i * nzh;
  const double kx = alpha * ((i < nx / 2) ? i : i - nx), kz = gamma * j;
  const double diag = (kx * kx + kz * kz) / re + inv_dt;
  double2* LU = ws + (size_t)blockIdx.x * ws_stride;
  double2* X = LU + (size_t)n4 * n4;
  double2* Rw = X + (size_t)n4 * C;
  for (int e = tid; e < n4 * n4; e += 256) {
    const int r = e / n4, c = e - r * n4;
    LU[e] = adv_entry(N, kx, kz, re, diag, r, c);
  }
  __syncthreads();
  bool singular = false;
  for (int k = 0; k < n4; ++k) {
    double best = -1.0;
    int bi = n4;
    for (int r = k + tid; r < n4; r += 256) {
      const double2 a = LU[(size_t)r * n4 + k];
      const double v = hypot(a.x, a.y);
      if (v > best) best = v, bi = r;
    }
    bval[tid] = best;
    bidx[tid] = bi;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) {
        const double o = bval[tid + h];
        const int oi = bidx[tid + h];
        if (o > bval[tid] || (o == bval[tid] && oi < bidx[tid])) bval[tid] = o, bidx[tid] = oi;
      }
      __syncthreads();
    }
    const int p = bidx[0];
    const double pv = bval[0];
    __syncthreads();
    if (!(pv > 0.0)) {
      singular = true;
      break;
    }
    if (tid == 0) piv[k] = p, nrows = 0;
    if (p != k)
      for (int c = tid; c < n4; c += 256) {
        const double2 t = LU[(size_t)k * n4 + c];
        LU[(size_t)k * n4 + c] = LU[(size_t)p * n4 + c];
        LU[(size_t)p * n4 + c] = t;
      }
    __syncthreads();
    const double2 akk = LU[(size_t)k * n4 + k];
    const double den = akk.x * akk.x + akk.y * akk.y;
    const double ir = akk.x / den, ii = -akk.y / den;
    // multipliers; the rows with a non-zero one are listed through an LDS
    // counter (their order does not change any result)
    for (int r = k + 1 + tid; r < n4; r += 256) {
      const double2 l = LU[(size_t)r * n4 + k];
      if (l.x != 0.0 || l.y != 0.0) {
        LU[(size_t)r * n4 + k] = make_double2(l.x * ir - l.y * ii, l.x * ii + l.y * ir);
        rows[atomicAdd(&nrows, 1)] = r;
      }
    }
    __syncthreads();
    const int w = n4 - k - 1;
    const int tot = nrows * w;
    for (int e = tid; e < tot; e += 256) {
      const int q = e / w;
      const int c = k + 1 + (e - q * w);
      const int r = rows[q];
      const double2 l = LU[(size_t)r * n4 + k];
      const double2 u = LU[(size_t)k * n4 + c];
      double2 a = LU[(size_t)r * n4 + c];
      a.x -= l.x * u.x - l.y * u.y;
      a.y -= l.x * u.y + l.y * u.x;
      LU[(size_t)r * n4 + c] = a;
    }
    __syncthreads();
  }
  if (singular) {
    if (tid == 0) status[blockIdx.x] = 1;
    return;
  }
  if (tid == 0) status[blockIdx.x] = 0;
  for (int c = tid; c < C; c += 256)
    adv_solve_refine(LU, piv, N, kx, kz, re, diag, C, R, X, Rw, c, Rp,
                     S + (size_t)(i * (nzh - 1) + j) * C * Rp);
}

}  // namespace

__global__ void k_narrow(const double* __restrict__ a, float* __restrict__ b, size_t n) {
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n;
       t += (size_t)gridDim.x * blockDim.x)
    b[t] = (float)a[t];
}

// The (0,0) mode's operator and wall response (host, the Helmholtz sweep of
// solve_core.h per unit right-hand side), then the FP32 copy of all operators used
// by the mixed-precision path.
static sp_status finish_adv(sp_plan* p) {
  const Dims& d = p->d;
  const int N = d.N, n1 = d.ny, nm = N - 1, Rp = (3 * n1 + 1) & ~1;
  std::vector<double> hw(3 * n1), blk(4 * n1 + 2), r(n1), q(n1), work(n1);
  rhs_weights(N, hw.data());
  sweep_factor(N, d.re * d.inv_dt, blk.data());
  const SweepView sw(blk.data(), n1);
  std::vector<double> S((size_t)3 * nm * Rp, 0.0), wall(n1, 0.0);
  for (int n = 0; n < nm; ++n) {
    std::fill(r.begin(), r.end(), 0.0);
    std::fill(q.begin(), q.end(), 0.0);
    r[n] = -d.re;
    sweep_solve<double>(sw, hw.data(), N, n & 1, r.data(), 0.0, q.data(), work.data());
    for (int c = 0; c < 3; c += 2)
      for (int m = n & 1; m <= N; m += 2) S[(size_t)(c * nm + n) * Rp + c * n1 + m] = q[m];
  }
  std::fill(r.begin(), r.end(), 0.0);
  for (int par = 0; par < 2; ++par) {
    const double beta = 0.5 * (par ? d.wall_upper - d.wall_lower : d.wall_upper + d.wall_lower);
    sweep_solve<double>(sw, hw.data(), N, par, r.data(), beta, wall.data(), work.data());
  }
  sp_status s = hip_check(p, hipMemcpy(p->d_adv, S.data(), S.size() * sizeof(double),
                                       hipMemcpyHostToDevice),
                          "upload the mean operator");
  if (s) return s;
  s = hip_check(p, hipMemcpy(p->d_advwall, wall.data(), n1 * sizeof(double), hipMemcpyHostToDevice),
                "upload the wall response");
  if (s) return s;
  hipLaunchKernelGGL(k_narrow, dim3(4096), dim3(256), 0, p->stream, p->d_adv, p->f_adv,
                     adv_count(p));
  s = hip_check(p, hipGetLastError(), "narrow operators");
  if (s) return s;
  return hip_check(p, hipStreamSynchronize(p->stream), "sync");
}

// Allocates the operators (FP64 and the FP32 copy) and the wall response if needed.
static sp_status ensure_adv_buffers(sp_plan* p) {
  auto get = [&](auto** q, size_t bytes) {
    if (*q || hipMalloc((void**)q, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *q = nullptr;
    return false;
  };
  if (!get(&p->d_adv, adv_count(p) * sizeof(double)) ||
      !get(&p->f_adv, adv_count(p) * sizeof(float)) ||
      !get(&p->d_advwall, p->d.ny * sizeof(double)))
    return set_error(p, SP_ERR_NOMEM, "cannot allocate the advected solve operators");
  return SP_OK;
}

// The operators of the modes in work built on the device (k_adv_build), in
// chunks whose scratch stays below 4 GiB (freed before returning);
// synchronises.
static sp_status build_advection_device(sp_plan* p, const std::vector<int>& work) {
  const Dims& d = p->d;
  const int N = d.N, n4 = 4 * d.ny, C = 3 * (N - 1);
  if (n4 > kAdvMaxN4) return set_error(p, SP_ERR_INVALID, "ny too large for the device build");
  sp_status s = ensure_adv_buffers(p);
  if (s) return s;
  s = hip_check(p, hipMemsetAsync(p->d_adv, 0, adv_count(p) * sizeof(double), p->stream), "clear operators");
  if (s) return s;
  if (work.empty()) {
    s = hip_check(p, hipStreamSynchronize(p->stream), "sync");
    return s ? s : finish_adv(p);
  }
  const size_t per_mode = (size_t)n4 * n4 + (size_t)2 * n4 * C;  // double2 entries
  const size_t cap = ((size_t)4 << 30) / (per_mode * sizeof(double2));
  const int chunk = (int)std::max<size_t>(1, std::min<size_t>(cap, work.size()));
  // scratch for the build only: the chunk's factors and columns, then the mode
  // list and status
  const size_t ws_bytes = (size_t)chunk * per_mode * sizeof(double2);
  void* scratch = nullptr;
  if (hipMalloc(&scratch, ws_bytes + (work.size() + chunk) * sizeof(int)) != hipSuccess) {
    (void)hipGetLastError();
    return set_error(p, SP_ERR_NOMEM, "cannot allocate the scratch of the advected build");
  }
  double2* ws = reinterpret_cast<double2*>(scratch);
  int* d_modes = reinterpret_cast<int*>(reinterpret_cast<char*>(scratch) + ws_bytes);
  int* d_status = d_modes + work.size();
  s = hip_check(p, hipMemcpy(d_modes, work.data(), work.size() * sizeof(int), hipMemcpyHostToDevice),
                "upload modes");
  std::vector<int> st(chunk);
  for (size_t off = 0; s == SP_OK && off < work.size(); off += chunk) {
    const int cnt = (int)std::min<size_t>(chunk, work.size() - off);
    hipLaunchKernelGGL(k_adv_build, dim3(cnt), dim3(256), 0, p->stream, d_modes + off, N, d.nx,
                       d.nzh, d.alpha, d.gamma, d.re, d.inv_dt, ws, per_mode, p->d_adv, d_status);
    s = hip_check(p, hipGetLastError(), "advected build");
    if (s) break;
    s = hip_check(p, hipMemcpyAsync(st.data(), d_status, cnt * sizeof(int), hipMemcpyDeviceToHost,
                                    p->stream),
                  "copy status");
    if (s) break;
    s = hip_check(p, hipStreamSynchronize(p->stream), "sync");
    for (int b = 0; s == SP_OK && b < cnt; ++b)
      if (st[b]) s = set_error(p, SP_ERR_INVALID, "singular advected tau system");
  }
  (void)hipStreamSynchronize(p->stream);  // no launch may still use the scratch
  (void)hipFree(scratch);
  if (s) return s;
  return finish_adv(p);
}

sp_status build_advection(sp_plan* p) {
  const Dims& d = p->d;
  const int N = d.N, C = 3 * (N - 1), R = 3 * d.ny, Rp = (R + 1) & ~1;
  std::vector<int> work;  // one mode of each pair (+-m_x, m_z); the mean mode apart
  for (int i = 0; i < d.nx / 2; ++i)
    for (int j = 0; j < d.nzm; ++j)
      if (i || j) work.push_back(i * d.nzh + j);
  if (!p->adv_host) return build_advection_device(p, work);
  using cplx = std::complex<double>;
  std::vector<double> S(adv_count(p), 0.0);
  unsigned nt = std::thread::hardware_concurrency();
  nt = std::max(1u, std::min(nt == 0 ? 1u : nt, 16u));
  std::vector<int> ok(nt, 1);
  std::vector<std::thread> th;
  for (unsigned t = 0; t < nt; ++t)
    th.emplace_back([&, t]() {
      std::vector<cplx> M((size_t)C * R);
      for (size_t w = t; w < work.size(); w += nt) {
        const int m = work[w];
        const int i = m / d.nzh, j = m - i * d.nzh;
        if (!adv_mode_operator(N, d.alpha * i, d.gamma * j, d.re, d.inv_dt, M.data())) {
          ok[t] = 0;
          continue;
        }
        double* o = &S[(size_t)(i * d.nzm + j) * C * Rp];
        for (int c = 0; c < C; ++c)
          for (int r = 0; r < R; ++r) {
            const cplx z = M[(size_t)c * R + r];
            o[(size_t)c * Rp + r] = adv_real_entry(z.real(), z.imag(), r % d.ny, c % (N - 1));
          }
      }
    });
  for (auto& x : th) x.join();
  for (int v : ok)
    if (!v) return set_error(p, SP_ERR_INVALID, "singular advected tau system");
  sp_status s = ensure_adv_buffers(p);
  if (s) return s;
  s = hip_check(p, hipMemcpy(p->d_adv, S.data(), S.size() * sizeof(double), hipMemcpyHostToDevice),
                "upload advected operators");
  if (s) return s;
  return finish_adv(p);
}

// g: NULL in FP64 (the analysis of p->nv is taken in the kernel).
template <bool RES>
static hipError_t adv_launch(sp_plan* p, const double2* g, const double2* x, double2* out,
                             int inhomogeneous, double oa, double ob, bool fp32) {
  const Dims& d = p->d;
  const int C = 3 * (d.N - 1), jh = d.N / 2 + 1;
  const size_t sh = (size_t)4 * C * sizeof(double) +
                    std::max<size_t>((size_t)12 * jh * sizeof(double2),
                                     (size_t)8 * kAdvRows * sizeof(double));
  const dim3 grid((d.nx / 2) * d.nzm + d.nzh + d.nx);
  const double* wall = inhomogeneous ? p->d_advwall : nullptr;
  SP_PROF_BEGIN(p, KID_ADV);
  if (fp32)
    hipLaunchKernelGGL((k_adv_apply<float, 0, RES>), grid, dim3(256), sh, p->stream, g, x,
                       d.inv_dt, p->f_adv, p->d_adv, wall, out, d.nx, d.ny, d.nzh, d.alpha,
                       (const double2*)nullptr, (const double*)nullptr, oa, ob);
  else
    hipLaunchKernelGGL((k_adv_apply<double, 1, RES>), grid, dim3(256), sh, p->stream, g, x,
                       d.inv_dt, p->d_adv, p->d_adv, wall, out, d.nx, d.ny, d.nzh, d.alpha,
                       (const double2*)p->nv, p->d_tinv_th, oa, ob);
  SP_PROF_END(p, KID_ADV);
  return hipGetLastError();
}

hipError_t launch_adv_solve(sp_plan* p, const double2* x, double2* out, int inhomogeneous,
                            bool fp32) {
  if (fp32) {
    const hipError_t e = launch_analysis_rhs(p, x, p->d.inv_dt, p->g, true);
    if (e != hipSuccess) return e;
  }
  return adv_launch<false>(p, p->g, x, out, inhomogeneous, 1.0, 0.0, fp32);
}

hipError_t launch_adv_solve_res(sp_plan* p, const double2* x, double oa, double ob, double2* out,
                                bool fp32) {
  if (fp32) {
    const hipError_t e = launch_analysis_rhs(p, x, p->d.inv_dt, p->g, true);
    if (e != hipSuccess) return e;
  }
  return adv_launch<true>(p, p->g, x, out, 0, oa, ob, fp32);
}

}  // namespace sp
