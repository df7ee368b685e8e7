// bssn_multipole.hip -- multipole coefficients of a complex grid function on
// a coordinate sphere (Einstein Toolkit paper, analysis section: the
// multipole module projects a field interpolated onto spheres onto
// spin-weighted spherical harmonics, C^lm = integral conj(sY_lm) u r^2 dOmega).
//
// Three launches, four for large spheres:
//   k_gl_nodes      (large spheres) the Gauss-Legendre nodes theta_j;
//   k_sphere_interp four threads per sphere point (theta_j, phi_k): the
//                   node theta_j where it is not there yet, and the tricubic
//                   interpolation of the real and imaginary parts (4 x 4 x 4
//                   storage points, block clamped into the grid);
//   k_multipole     one workgroup per (l, m, chunk of the points): the sum
//                   of conj(sY_lm) u w_j (2 pi / n_phi) over its points, a
//                   fixed-order tree reduction;
//   k_multipole_sum one thread per (l, m): the chunks added in order (the
//                   result is deterministic), times r^2.
// sY_lm (Goldberg's sum) is evaluated with half-angle powers,
//   sin^{2l-k}(theta/2) cos^{k}(theta/2), k = 2r + s - m in [0, 2l],
// so no cotangent is formed.
// A sphere is a few thousand points, so every launch is bound by the latency
// of its serial chains, not by memory.  64 x 128 points with l <= 8: 26 us a
// call in a row of calls (33 us of kernels in a trace), against 58 (74) when the
// nodes were a launch of their own with a division per recurrence step (22 in
// the trace), the interpolation took one thread per point (25) and every point
// formed its binomials (21).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bssn_internal.h"
#include "bssn_kernels.h"

namespace bssn {
namespace {

__device__ __forceinline__ double ipow(double x, int n) {
  double r = 1.0;
  while (n > 0) {
    if (n & 1) r *= x;
    x *= x;
    n >>= 1;
  }
  return r;
}

__device__ __forceinline__ double fact(int n) {
  double r = 1.0;
  for (int k = 2; k <= n; ++k) r *= k;
  return r;
}

__device__ __forceinline__ double binom(int n, int k) {
  if (k < 0 || k > n) return 0.0;
  double r = 1.0;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

// P_n(z) in p1 and P_{n-1}(z) in p0, rec[k] = {(2k - 1)/k, (k - 1)/k}: with the
// divisions in the table the chain of a step is one FMA.
__device__ __forceinline__ void legendre(const double2* rec, int n, double z,
                                         double& p0, double& p1) {
  p0 = 1.0;
  p1 = z;
#pragma unroll 4
  for (int k = 2; k <= n; ++k) {
    const double2 c = rec[k];
    const double p2 = c.x * z * p1 - c.y * p0;
    p0 = p1;
    p1 = p2;
  }
}

// Gauss-Legendre node j of n (ascending in x = cos(theta)) and its weight, by
// Newton iteration on the Legendre recurrence.
__device__ __forceinline__ void gl_node(const double2* rec, int n, int j,
                                        double& x, double& w) {
  const int jd = n - 1 - j;  // the guess below is descending in j
  double z = cos(M_PI * (jd + 0.75) / (n + 0.5));
  double p0, p1;
  for (int it = 0; it < 100; ++it) {
    legendre(rec, n, z, p0, p1);
    const double dp = n * (z * p1 - p0) / (z * z - 1.0);
    const double dz = p1 / dp;
    z -= dz;
    if (fabs(dz) <= 1e-15 * fabs(z)) break;  // dz = 0 at the middle node
  }
  // the weight from the derivative at the converged node
  legendre(rec, n, z, p0, p1);
  const double dp = n * (z * p1 - p0) / (z * z - 1.0);
  x = z;
  w = 2.0 / ((1.0 - z * z) * dp * dp);
}

// The recurrence's ratios up to n, by the nt threads of a workgroup.
__device__ __forceinline__ void fill_ratios(double2* rec, int n, int nt) {
  for (int k = 2 + threadIdx.x; k <= n; k += nt)
    rec[k] = {(2.0 * k - 1.0) / k, (k - 1.0) / k};
  __syncthreads();
}

// The nodes by themselves, one per thread.
__global__ void __launch_bounds__(64)
    k_gl_nodes(const int n, double* __restrict__ xs, double* __restrict__ ws) {
  extern __shared__ double2 rec[];
  fill_ratios(rec, n, 64);
  const int j = blockIdx.x * 64 + threadIdx.x;
  if (j >= n) return;
  double x, w;
  gl_node(rec, n, j, x, w);
  xs[j] = x;
  ws[j] = w;
}

// Lane q of a point's four takes the z plane q of its 4 x 4 x 4 block, so its
// 32 loads are in flight together.  NODES: each point works out its own node
// and the first of a row leaves it for the next launch; else the nodes are
// there (launch_multipole has the rule).
template <bool NODES>
__global__ void __launch_bounds__(256)
    k_sphere_interp(const MultipoleArgs A, double* __restrict__ xs,
                    double* __restrict__ ws, double* __restrict__ val) {
  extern __shared__ double2 rec[];
  if constexpr (NODES) fill_ratios(rec, A.ntheta, 256);
  const int p = (blockIdx.x * 256 + threadIdx.x) >> 2, kk = threadIdx.x & 3;
  if (p >= A.ntheta * A.nphi) return;
  const int j = p / A.nphi, k = p % A.nphi;
  double ct;
  if constexpr (NODES) {
    double wj;
    gl_node(rec, A.ntheta, j, ct, wj);
    if (k == 0 && kk == 0) {
      xs[j] = ct;
      ws[j] = wj;
    }
  } else {
    ct = xs[j];
  }
  const double st = sqrt(fmax(0.0, 1.0 - ct * ct));
  const double ph = 2.0 * M_PI * k / A.nphi;
  const double pos[3] = {A.centre[0] + A.radius * st * cos(ph),
                         A.centre[1] + A.radius * st * sin(ph),
                         A.centre[2] + A.radius * ct};
  const int g = A.ghost;
  double wt[3][4];
  int b[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int N = A.n[a] + 2 * g;
    const double s = (pos[a] - (A.origin[a] - g * A.h[a])) / A.h[a];
    double fs = floor(s);
    if (!(fs >= -2.0)) fs = -2.0;  // also NaN
    if (fs > double(N)) fs = double(N);
    int bb = int(fs) - 1;
    bb = bb < 0 ? 0 : (bb > N - 4 ? N - 4 : bb);
    b[a] = bb;
    const double t = s - bb;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      double q = 1.0;
#pragma unroll
      for (int l = 0; l < 4; ++l)
        if (l != m) q *= (t - l) / double(m - l);
      wt[a][m] = q;
    }
  }
  double re = 0.0, im = 0.0;
  const int64_t base =
      int64_t(b[2] + kk) * A.sz + int64_t(b[1]) * A.sy + b[0];
  const double wz = kk == 0   ? wt[2][0]
                    : kk == 1 ? wt[2][1]
                    : kk == 2 ? wt[2][2]
                              : wt[2][3];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      const double w = wz * wt[1][jj] * wt[0][ii];
      const int64_t o = base + jj * A.sy + ii;
      re += w * A.re[o];
      if (A.im) im += w * A.im[o];
    }
#pragma unroll
  for (int h = 1; h < 4; h *= 2) {
    re += __shfl_xor(re, h, 64);
    im += __shfl_xor(im, h, 64);
  }
  if (kk == 0) {
    val[2 * p] = re;
    val[2 * p + 1] = im;
  }
}

// With r from r0 to r1 the powers in Goldberg's sum step by cos^2 up and sin^2
// down, so a point's sum is a homogeneous Horner scheme over coefficients that
// the workgroup forms once (r1 - r0 <= l - max(|m|, |s|) and l <= 16 by the entry
// point's check, so there are at most 17).
__global__ void __launch_bounds__(256)
    k_multipole(const MultipoleArgs A, const double* __restrict__ x,
                const double* __restrict__ w, const double* __restrict__ val,
                const int nchunk, double* __restrict__ part) {
  __shared__ double coef[32], red[2][4];
  const int q = blockIdx.x / nchunk, chunk = blockIdx.x % nchunk;
  const int t = threadIdx.x;
  int l = 0;
  while ((l + 1) * (l + 1) <= q) ++l;
  const int m = q - l * l - l;
  const int s = A.spin;
  double are = 0.0, aim = 0.0;
  if (l >= (s < 0 ? -s : s)) {
    const int r0 = m - s > 0 ? m - s : 0;
    const int r1 = l - s < l + m ? l - s : l + m;
    if (t <= r1 - r0) {
      const int r = r0 + t;
      const double pre =
          ((m & 1) ? -1.0 : 1.0) *
          sqrt(fact(l + m) * fact(l - m) * (2 * l + 1) /
               (4.0 * M_PI * fact(l + s) * fact(l - s)));
      const double sign = ((l - r - s) & 1) ? -1.0 : 1.0;
      coef[t] = pre * sign * binom(l - s, r) * binom(l + s, r + s - m);
    }
    __syncthreads();
    const double dphi = 2.0 * M_PI / A.nphi;
    const int npts = A.ntheta * A.nphi;
    const int elo = 2 * r0 + s - m, ehi = 2 * l - (2 * r1 + s - m);
    for (int p = chunk * 256 + t; p < npts; p += nchunk * 256) {
      const int j = p / A.nphi, k = p % A.nphi;
      const double ct = x[j];
      const double s2 = fmax(0.0, 0.5 * (1.0 - ct));
      const double c2 = fmax(0.0, 0.5 * (1.0 + ct));
      double y = coef[0], cp = 1.0;
      for (int i = 1; i <= r1 - r0; ++i) {
        cp *= c2;
        y = y * s2 + coef[i] * cp;
      }
      // real part of sY_lm without e^{i m phi}
      y *= ipow(sqrt(s2), ehi) * ipow(sqrt(c2), elo);
      double sn, cs;
      sincos(m * (dphi * k), &sn, &cs);
      // conj(Y) u = y (cos - i sin)(u_re + i u_im)
      const double ur = val[2 * p], ui = val[2 * p + 1];
      const double wq = w[j] * dphi;
      are += wq * y * (cs * ur + sn * ui);
      aim += wq * y * (cs * ui - sn * ur);
    }
  }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) {
    are += __shfl_xor(are, h, 64);
    aim += __shfl_xor(aim, h, 64);
  }
  if ((t & 63) == 0) {
    red[0][t >> 6] = are;
    red[1][t >> 6] = aim;
  }
  __syncthreads();
  if (t < 2)
    part[2 * (q * nchunk + chunk) + t] =
        (red[t][0] + red[t][1]) + (red[t][2] + red[t][3]);
}

// One thread per (l, m): the chunks' partial sums added in chunk order.
__global__ void __launch_bounds__(64)
    k_multipole_sum(const int nq, const int nchunk, const double radius,
                    const double* __restrict__ part,
                    double* __restrict__ coeffs) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nq) return;
  double re = 0.0, im = 0.0;
#pragma unroll 8
  for (int c = 0; c < nchunk; ++c) {
    re += part[2 * (q * nchunk + c)];
    im += part[2 * (q * nchunk + c) + 1];
  }
  coeffs[2 * q] = re * radius * radius;
  coeffs[2 * q + 1] = im * radius * radius;
}

// Whether each sphere point works out its own node (no launch more).  That takes
// one Newton iteration per wave, as long as one iteration in a launch of its own
// while the waves of a SIMD fill each other's waits; beyond two per SIMD (32,768
// points) they queue, and the redundant recurrence steps, points x ntheta of them
// per iteration, come to cost more than a launch does.  Both ways, own nodes first
// (us per call, l <= 8): 64 x 128 26 and 27, 512 x 64 83 and 87, 180 x 266 66 and
// 67, 360 x 100 79 and 76, 256 x 512 152 and 129, 1024 x 128 343 and 198,
// 1024 x 4096 9,040 and 2,760.
inline bool own_nodes(int ntheta, int npts) {
  return npts <= 32768 || int64_t(npts) * ntheta <= 1 << 23;
}
}  // namespace

hipError_t launch_multipole(const MultipoleArgs& A, double* work,
                            double* coeffs, hipStream_t st) {
  double* x = work;
  double* w = work + A.ntheta;
  double* val = work + 2 * A.ntheta;
  const int npts = A.ntheta * A.nphi;
  const size_t ratios = sizeof(double2) * (A.ntheta + 1);
  const dim3 grd((npts + 63) / 64);
  hipError_t e;
  if (own_nodes(A.ntheta, npts)) {
    hipLaunchKernelGGL(k_sphere_interp<true>, grd, dim3(256), ratios, st, A, x,
                       w, val);
  } else {
    hipLaunchKernelGGL(k_gl_nodes, dim3((A.ntheta + 63) / 64), dim3(64),
                       ratios, st, A.ntheta, x, w);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sphere_interp<false>, grd, dim3(256), 0, st, A, x, w,
                       val);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nq = (A.lmax + 1) * (A.lmax + 1);
  // four points per thread repay forming the coefficients; never more chunks
  // than the workspace has room for
  const int nchunk =
      std::min((npts + 1023) / 1024, multipole_chunks(A.ntheta, A.nphi));
  double* part = val + 2 * int64_t(npts);
  hipLaunchKernelGGL(k_multipole, dim3(nq * nchunk), dim3(256), 0, st, A, x,
                     w, val, nchunk, part);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_multipole_sum, dim3((nq + 63) / 64), dim3(64), 0, st,
                     nq, nchunk, A.radius, part, coeffs);
  return hipGetLastError();
}

}  // namespace bssn
