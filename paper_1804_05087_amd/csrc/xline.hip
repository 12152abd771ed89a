// x-line kernels with register-resident FFTs (paper Sec. 3.2: 3/2 zero
// padding in x). Same four-step split as the z-line kernels: a line of length
// P = P1 * P2 is transformed by P2 threads holding P1 values each, one
// exchange through LDS, then P1 threads holding P2 values each.
//
//   k_xinv_reg  y-valued spectral fields [f][y][kz][mx] (nx modes, FFT order)
//               -> zero padded to P = 3 nx / 2 -> inverse FFT -> [f][y][x][kz]
//   k_xfwd_reg  [f][y][x][kz] -> forward FFT -> truncated to nx modes (Nyquist
//               zero) -> [f][y][kz][mx]
// Block: (y, field, chunk of kc z-modes); a thread of the second step writes
// its physical points for consecutive kz, so stores to the x-major layout are
// contiguous across lanes.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "sp_internal.h"

namespace sp {

// Logical block (y, field, z-chunk) of an x-line grid (hardware grid
// (ny, nfields, chunks)), reordered by xcd_order with the field fastest and
// then the chunk: the blocks of one (y, chunk), which read the same spectral
// lines for different output fields, share an L2.
// MB: the grid's first dimension counts the planes of every member of a batch.
struct XBlk {
  int member, y, f, ch;
};
template <bool MB>
__device__ inline XBlk xline_block(int ny) {
  const int gy = gridDim.x, gf = gridDim.y, gc = gridDim.z;
  const int b = blockIdx.x + gy * (blockIdx.y + gf * blockIdx.z);
  const int l = xcd_order(b, gy * gf * gc);
  const int my = l / (gf * gc);
  const int member = MB ? my / ny : 0;
  return XBlk{member, my - member * ny, l % gf, (l / gf) % gc};
}

// Modes per block of the FP64 inverse transform (128 threads): a thread takes one column
// of step 1 and at most xinv_passes columns of step 2, since the columns stay in registers
// while their real parts, then their imaginary ones, go through LDS. Bound by how many
// waves hide the chains of the transforms: with half the LDS a CU holds eight blocks
// instead of five, and the six fields take 27.1 us instead of 34.7 at 96x97x96, 25.9
// instead of 33.5 at 128x49x128, 11.0 as before at 72x49x72. FP32 lines are half as long
// in LDS already and keep the exchange in one piece.
__host__ __device__ constexpr int xinv_passes(int P1, int P2) { return 2 * P1 > 3 * P2 ? 2 : 1; }
constexpr int xinv_max_modes(int P1, int P2) {
  const int a = 128 / P2, b = 128 * xinv_passes(P1, P2) / P1;
  return a < b ? a : b;
}

// plain == 0: output field f of (u, v, w, omega_x, omega_y, omega_z) from the
// five y-valued fields (u, du/dy, v, w, dw/dy) with i k_x, i k_z; plain != 0:
// output field f is input field f.
template <typename R, int P1, int P2, bool MB>
__global__ void __launch_bounds__(128)
    k_xinv_reg(const typename V2<R>::T* __restrict__ yv, typename V2<R>::T* __restrict__ xp,
               const typename V2<R>::T* __restrict__ tw, int nx, int ny, int nzm, int kc, R alpha,
               R gamma, int plain, size_t mi, size_t mo) {
  using C = typename V2<R>::T;
  constexpr int P = P1 * P2;
  constexpr int S1 = P1 + 1;
  extern __shared__ unsigned char smem_raw[];
  C* twl = reinterpret_cast<C*>(smem_raw);
  const XBlk bk = xline_block<MB>(ny);
  if constexpr (MB) {
    yv += bk.member * mi;
    xp += bk.member * mo;
  }
  const int y = bk.y;
  const int f = bk.f;
  const int kz0 = bk.ch * kc;
  const int nl = min(kc, nzm - kz0);
  for (int t = threadIdx.x; t < P; t += blockDim.x) twl[t] = tw[t];
  __syncthreads();
  const size_t fs = (size_t)ny * nzm * nx;
  const int h = nx / 2;
  // step 1: task (l, n2), values at padded positions pos = P2 n1 + n2; then the exchange
  // and step 2: task (k1, l), physical points x = k1 + P1 k2
  C* dst = xp + ((size_t)f * ny + y) * P * nzm + kz0;
  auto step1 = [&](int l, int n2, C(&v)[P1]) {
    const int kz = kz0 + l;
    const C* src = yv + ((size_t)y * nzm + kz) * nx;
    const R kzv = gamma * (R)kz;
#pragma unroll
    for (int n1 = 0; n1 < P1; ++n1) {
      // positions of the padding alone (four of sixteen) are not loaded: 27.1 -> 25.0 us
      // at 96x97x96, 11.0 -> 9.8 at 72x49x72
      if (P2 * n1 >= P / 3 && P2 * n1 + P2 - 1 <= P - P / 3) {
        v[n1] = mk((R)0, (R)0);
        continue;
      }
      const int pos = P2 * n1 + n2;
      const bool lo = P2 * n1 + P2 <= P / 3 || pos < h;
      const bool hi = P2 * n1 > P - P / 3 || pos > P - h;
      const int i = lo ? pos : (hi ? pos - P + nx : 0);
      const R keep = (lo || hi) ? (R)1 : (R)0;
      const R kxv = alpha * (R)(lo ? i : i - nx);
      C val;
      if (plain) {
        val = src[f * fs + i];
      } else if (f == 0) {
        val = src[i];
      } else if (f == 1) {
        val = src[2 * fs + i];
      } else if (f == 2) {
        val = src[3 * fs + i];
      } else if (f == 3) {  // dw/dy - i kz v
        val = csub(src[4 * fs + i], sidot(cscale(src[2 * fs + i], kzv), (R)1));
      } else if (f == 4) {  // i kz u - i kx w
        val = sidot(csub(cscale(src[i], kzv), cscale(src[3 * fs + i], kxv)), (R)1);
      } else {  // i kx v - du/dy
        val = csub(sidot(cscale(src[2 * fs + i], kxv), (R)1), src[fs + i]);
      }
      v[n1] = cscale(val, keep);
    }
    dft_reg<P1, P, C, R>(v, (R)1, twl);
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      if (n2 != 0) v[k1] = cmul(v[k1], wpow<P, P, C, R>(n2 * k1, (R)1, twl));
  };
  auto step2 = [&](int k1, int l, C(&t)[P2]) {
    dft_reg<P2, P, C, R>(t, (R)1, twl);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) dst[(size_t)(k1 + P1 * k2) * nzm + l] = t[k2];
  };
  if constexpr (sizeof(R) == 8) {
    R* ex = reinterpret_cast<R*>(twl + P);  // [kc][P2][S1]
    constexpr int NP = xinv_passes(P1, P2);
    const int l1 = threadIdx.x / P2;
    const int n2 = threadIdx.x - l1 * P2;
    const bool act = l1 < kc && l1 < nl;  // kc P2 <= 128: one task a thread
    C v[P1], t[NP][P2];
    if (act) step1(l1, n2, v);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      if (part) __syncthreads();
      if (act) {
        R* e = ex + (l1 * P2 + n2) * S1;
#pragma unroll
        for (int k1 = 0; k1 < P1; ++k1) e[k1] = part ? v[k1].y : v[k1].x;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int task = threadIdx.x + 128 * q;
        const int k1 = task / kc;
        const int l = task - k1 * kc;
        if (k1 < P1 && l < nl) {
          const R* e = ex + l * P2 * S1 + k1;
#pragma unroll
          for (int m = 0; m < P2; ++m) (part ? t[q][m].y : t[q][m].x) = e[m * S1];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int task = threadIdx.x + 128 * q;
      const int k1 = task / kc;
      const int l = task - k1 * kc;
      if (k1 < P1 && l < nl) step2(k1, l, t[q]);
    }
  } else {
    // FP32 keeps the one exchange and every rounding: which products the compiler contracts
    // into fused multiply-adds follows the code's shape
    C* ex = twl + P;  // [kc][P2][S1]
    // step 1: task (l, n2), values at padded positions pos = P2 n1 + n2
    for (int task = threadIdx.x; task < kc * P2; task += blockDim.x) {
      const int l = task / P2;
      const int n2 = task - l * P2;
      if (l < nl) {
        const int kz = kz0 + l;
        const C* src = yv + ((size_t)y * nzm + kz) * nx;
        const R kzv = gamma * (R)kz;
        C v[P1];
#pragma unroll
        for (int n1 = 0; n1 < P1; ++n1) {
          const int pos = P2 * n1 + n2;
          const bool lo = pos < h;
          const bool hi = pos > P - h;
          const int i = lo ? pos : (hi ? pos - P + nx : 0);
          const R keep = (lo || hi) ? (R)1 : (R)0;
          const R kxv = alpha * (R)(lo ? i : i - nx);
          C val;
          if (plain) {
            val = src[f * fs + i];
          } else if (f == 0) {
            val = src[i];
          } else if (f == 1) {
            val = src[2 * fs + i];
          } else if (f == 2) {
            val = src[3 * fs + i];
          } else if (f == 3) {  // dw/dy - i kz v
            val = csub(src[4 * fs + i], sidot(cscale(src[2 * fs + i], kzv), (R)1));
          } else if (f == 4) {  // i kz u - i kx w
            val = sidot(csub(cscale(src[i], kzv), cscale(src[3 * fs + i], kxv)), (R)1);
          } else {  // i kx v - du/dy
            val = csub(sidot(cscale(src[2 * fs + i], kxv), (R)1), src[fs + i]);
          }
          v[n1] = cscale(val, keep);
        }
        dft_reg<P1, P, C, R>(v, (R)1, twl);
        C* e = ex + (l * P2 + n2) * S1;
#pragma unroll
        for (int k1 = 0; k1 < P1; ++k1)
          e[k1] = (k1 == 0 || n2 == 0) ? v[k1] : cmul(v[k1], wpow<P, P, C, R>(n2 * k1, (R)1, twl));
      }
    }
    __syncthreads();
    // step 2: task (k1, l), physical points x = k1 + P1 k2
    for (int task = threadIdx.x; task < P1 * kc; task += blockDim.x) {
      const int k1 = task / kc;
      const int l = task - k1 * kc;
      if (l < nl) {
        C t[P2];
        const C* e = ex + l * P2 * S1 + k1;
#pragma unroll
        for (int n2 = 0; n2 < P2; ++n2) t[n2] = e[n2 * S1];
        dft_reg<P2, P, C, R>(t, (R)1, twl);
#pragma unroll
        for (int k2 = 0; k2 < P2; ++k2) dst[(size_t)(k1 + P1 * k2) * nzm + l] = t[k2];
      }
    }
  }
}

// SB (the SBDF2 steps' extrapolation, taken as the result is stored): nv = 2 v - prev
// and prev = v with v the transform, prev in nv's layout; first: nv = prev = v.
template <typename R, int P1, int P2, bool MB, bool SB = false>
__global__ void __launch_bounds__(128)
    k_xfwd_reg(const typename V2<R>::T* __restrict__ np, typename V2<R>::T* __restrict__ nv,
               const typename V2<R>::T* __restrict__ tw, int nx, int ny, int nzm, int kc, size_t mi,
               size_t mo, typename V2<R>::T* __restrict__ prev = nullptr, int first = 0) {
  using C = typename V2<R>::T;
  constexpr int P = P1 * P2;
  constexpr int S1 = P1 + 1;
  extern __shared__ unsigned char smem_raw[];
  C* twl = reinterpret_cast<C*>(smem_raw);
  C* ex = twl + P;  // [kc][P2][S1]
  const XBlk bk = xline_block<MB>(ny);
  if constexpr (MB) {
    np += bk.member * mi;
    nv += bk.member * mo;
  }
  const int y = bk.y;
  const int c = bk.f;
  const int kz0 = bk.ch * kc;
  const int nl = min(kc, nzm - kz0);
  for (int t = threadIdx.x; t < P; t += blockDim.x) twl[t] = tw[t];
  __syncthreads();
  const int h = nx / 2;
  // step 1: task (n1, l); points x = n1 + P1 n2, m = P2 m1 + m2
  const C* src = np + ((size_t)c * ny + y) * P * nzm + kz0;
  for (int task = threadIdx.x; task < P1 * kc; task += blockDim.x) {
    const int n1 = task / kc;
    const int l = task - n1 * kc;
    if (l < nl) {
      C t[P2];
#pragma unroll
      for (int n2 = 0; n2 < P2; ++n2) t[n2] = src[(size_t)(n1 + P1 * n2) * nzm + l];
      dft_reg<P2, P, C, R>(t, (R)-1, twl);
      C* e = ex + l * P2 * S1 + n1;
#pragma unroll
      for (int m2 = 0; m2 < P2; ++m2)
        e[m2 * S1] = (m2 == 0 || n1 == 0) ? t[m2] : cmul(t[m2], wpow<P, P, C, R>(n1 * m2, (R)-1, twl));
    }
  }
  __syncthreads();
  // step 2: task (l, m2); keep |m_x| < nx / 2
  for (int task = threadIdx.x; task < kc * P2; task += blockDim.x) {
    const int l = task / P2;
    const int m2 = task - l * P2;
    if (l < nl) {
      C v[P1];
      const C* e = ex + (l * P2 + m2) * S1;
#pragma unroll
      for (int n1 = 0; n1 < P1; ++n1) v[n1] = e[n1];
      dft_reg<P1, P, C, R>(v, (R)-1, twl);
      const size_t o = (((size_t)c * ny + y) * nzm + kz0 + l) * nx;
      C* dst = nv + o;
      if constexpr (SB) {
        C* pr = prev + o;
        C b[P1];
        if (!first) {  // uniform: every load in flight before the first store
#pragma unroll
          for (int m1 = 0; m1 < P1; ++m1) {
            const int pos = P2 * m1 + m2;
            const int i = pos < h ? pos : (pos > P - h ? pos - P + nx : 0);
            b[m1] = pr[i];
          }
        }
#pragma unroll
        for (int m1 = 0; m1 < P1; ++m1) {
          const int pos = P2 * m1 + m2;
          if (pos < h || pos > P - h) {
            const int i = pos < h ? pos : pos - P + nx;
            dst[i] = first ? v[m1] : mk((R)2 * v[m1].x - b[m1].x, (R)2 * v[m1].y - b[m1].y);
            pr[i] = v[m1];
          }
        }
      } else {
#pragma unroll
        for (int m1 = 0; m1 < P1; ++m1) {
          const int pos = P2 * m1 + m2;
          if (pos < h)
            dst[pos] = v[m1];
          else if (pos > P - h)
            dst[pos - P + nx] = v[m1];
        }
      }
      if (m2 == 0) dst[h] = mk((R)0, (R)0);
    }
  }
}

// ----------------------------------- launchers -----------------------------------

hipError_t launch_fft_x_inv_lds(sp_plan* p, const void* in, void* out, int nfields, int plain,
                                bool fp32);
hipError_t launch_fft_x_fwd_lds(sp_plan* p, const void* in, void* out, int nfields, bool fp32);

// z-modes per block: the fewest chunks that give the grid at least 512 blocks
// (and at least 4 modes per chunk) and keep the exchange buffer within 32 KiB (16 in
// FP32) of LDS or, exchanged in halves, within xinv_max_modes, split evenly; a chunk is
// widened to a whole number of 128-byte cache lines (8 FP64 or 16 FP32 complex values)
// when that keeps the same even split, so that chunks of the x-physical rows [x][kz]
// start on line boundaries. The LDS bound leaves a CU five blocks of two waves; with
// 64 KiB it had two, and the long lines waited: forward at 96x97x96 18.4 us (64 KiB),
// 11.8 (32), 12.1 (24), 13.5 (16); 128x49x128 17.2 / 11.0 / 12.3 / 12.0; FP32 inverse at
// 72x49x72 12.8 us (32 and 64 KiB), 8.9 (16).
static int xline_chunk(const Dims& d, int nb, int nfields, bool fp32, int P1, int P2,
                       bool halves = false) {
  const int lw = fp32 ? 16 : 8;
  const size_t el = fp32 ? sizeof(float2) : sizeof(double2);
  const long per = (long)d.ny * nfields * nb;
  const int nmax = d.nzm / 4 > 1 ? d.nzm / 4 : 1;
  const int most = halves ? xinv_max_modes(P1, P2) : d.nzm;
  auto over = [&](int kc) {
    return kc > most ||
           (!halves && ((size_t)d.px + (size_t)kc * P2 * (P1 + 1)) * el > (fp32 ? 16384 : 32768));
  };
  int nch = 1;
  while (nch < d.nzm && ((nch < nmax && per * nch < 512) || over((d.nzm + nch - 1) / nch))) ++nch;
  int kc = (d.nzm + nch - 1) / nch;
  const int ka = (kc + lw - 1) / lw * lw;
  if (d.nzm % ka == 0 && d.nzm / ka == nch && ka <= most) kc = ka;
  return kc;
}

hipError_t launch_fft_x_inv_gen(sp_plan* p, const void* in, void* out, int nfields, int plain,
                                bool fp32) {
  const Dims& d = p->d;
  const int P1 = reg_fft_split(d.px, fp32);
  if (P1 == 0) return launch_fft_x_inv_lds(p, in, out, nfields, plain, fp32);
  const int P2 = d.px / P1;
  const int kc = xline_chunk(d, p->mem.nb, nfields, fp32, P1, P2, !fp32);
  const dim3 grid(d.ny * p->mem.nb, nfields, (d.nzm + kc - 1) / kc);
  const size_t ex = (size_t)kc * P2 * (P1 + 1);
  const size_t sh = fp32 ? (d.px + ex) * sizeof(float2) : d.px * sizeof(double2) + ex * sizeof(double);
  SP_PROF_BEGIN(p, KID_FFT_X_INV);
#define XI32(A, B)                                                                              \
  hipLaunchKernelGGL((k_xinv_reg<float, A, B, MB>), grid, dim3(128), sh, p->stream,             \
                     (const float2*)in, (float2*)out, p->f_twx, d.nx, d.ny, d.nzm, kc,          \
                     (float)d.alpha, (float)d.gamma, plain, p->mem.yv, p->mem.xp)
#define XI64(A, B)                                                                              \
  hipLaunchKernelGGL((k_xinv_reg<double, A, B, MB>), grid, dim3(128), sh, p->stream,            \
                     (const double2*)in, (double2*)out, p->d_twx, d.nx, d.ny, d.nzm, kc,        \
                     d.alpha, d.gamma, plain, p->mem.yv, p->mem.xp)
  auto run = [&](auto mb) {
    constexpr bool MB = decltype(mb)::value;
    if (fp32) {
      SP_REG_FFT_DISPATCH(d.px, XI32)
    } else {
      SP_REG_FFT_DISPATCH64(d.px, XI64)
    }
  };
  if (p->mem.nb > 1)
    run(std::true_type{});
  else
    run(std::false_type{});
#undef XI32
#undef XI64
  SP_PROF_END(p, KID_FFT_X_INV);
  return hipGetLastError();
}

hipError_t launch_fft_x_fwd_gen(sp_plan* p, const void* in, void* out, int nfields, bool fp32) {
  const Dims& d = p->d;
  const int P1 = reg_fft_split(d.px, fp32);
  if (P1 == 0) return launch_fft_x_fwd_lds(p, in, out, nfields, fp32);
  const int P2 = d.px / P1;
  const int kc = xline_chunk(d, p->mem.nb, nfields, fp32, P1, P2);
  const dim3 grid(d.ny * p->mem.nb, nfields, (d.nzm + kc - 1) / kc);
  const size_t el = fp32 ? sizeof(float2) : sizeof(double2);
  const size_t sh = ((size_t)d.px + (size_t)kc * P2 * (P1 + 1)) * el;
  SP_PROF_BEGIN(p, KID_FFT_X_FWD);
#define XF32(A, B)                                                                              \
  hipLaunchKernelGGL((k_xfwd_reg<float, A, B, MB>), grid, dim3(128), sh, p->stream,             \
                     (const float2*)in, (float2*)out, p->f_twx, d.nx, d.ny, d.nzm, kc,          \
                     p->mem.np, p->mem.nv)
#define XF64(A, B)                                                                              \
  hipLaunchKernelGGL((k_xfwd_reg<double, A, B, MB>), grid, dim3(128), sh, p->stream,            \
                     (const double2*)in, (double2*)out, p->d_twx, d.nx, d.ny, d.nzm, kc,        \
                     p->mem.np, p->mem.nv)
  auto run = [&](auto mb) {
    constexpr bool MB = decltype(mb)::value;
    if (fp32) {
      SP_REG_FFT_DISPATCH(d.px, XF32)
    } else {
      SP_REG_FFT_DISPATCH64(d.px, XF64)
    }
  };
  if (p->mem.nb > 1)
    run(std::true_type{});
  else
    run(std::false_type{});
#undef XF32
#undef XF64
  SP_PROF_END(p, KID_FFT_X_FWD);
  return hipGetLastError();
}

// The forward x transform of a step's product fields with the SBDF2 extrapolation
// (FP64): p->nv = 2 N - prev, prev = N (first: both N). A launch of its own for it took
// 2.4 us of a 27 us step at 32x33x32.
hipError_t launch_fft_x_fwd_sbdf2(sp_plan* p, double2* prev, bool first) {
  const Dims& d = p->d;
  const int P1 = reg_fft_split(d.px, false);
  if (P1 == 0) {
    const hipError_t e = launch_fft_x_fwd_lds(p, p->np, p->nv, 3, false);
    if (e != hipSuccess) return e;
    return launch_sbdf2_combine(p, (double2*)p->nv, prev, (size_t)3 * d.ny * d.nzm * d.nx, first);
  }
  const int P2 = d.px / P1;
  const int kc = xline_chunk(d, 1, 3, false, P1, P2);
  const dim3 grid(d.ny, 3, (d.nzm + kc - 1) / kc);
  const size_t sh = ((size_t)d.px + (size_t)kc * P2 * (P1 + 1)) * sizeof(double2);
  SP_PROF_BEGIN(p, KID_FFT_X_FWD);
#define XS(A, B)                                                                               \
  hipLaunchKernelGGL((k_xfwd_reg<double, A, B, false, true>), grid, dim3(128), sh, p->stream,  \
                     (const double2*)p->np, (double2*)p->nv, p->d_twx, d.nx, d.ny, d.nzm, kc,  \
                     (size_t)0, (size_t)0, prev, first ? 1 : 0)
  SP_REG_FFT_DISPATCH64(d.px, XS)
#undef XS
  SP_PROF_END(p, KID_FFT_X_FWD);
  return hipGetLastError();
}

hipError_t launch_fft_x_inv(sp_plan* p, bool fp32) {
  return launch_fft_x_inv_gen(p, p->yv, p->xp, 6, 0, fp32);
}

hipError_t launch_fft_x_fwd(sp_plan* p, bool fp32) {
  return launch_fft_x_fwd_gen(p, p->np, p->nv, 3, fp32);
}

}  // namespace sp
