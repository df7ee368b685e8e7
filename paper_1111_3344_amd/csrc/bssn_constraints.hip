// bssn_constraints.hip -- Hamiltonian, momentum and conformal-connection
// constraints in FP64, with deterministic norms.
//
// H = R - K^i_j K^j_i + K^2 and M_i = D_j K^j_i - D_i K (vacuum; Einstein
// Toolkit paper, "Other analysis modules") written in the BSSN variables
// under the algebraic conditions det gt = 1 and tr A~ = 0:
//   R   = e^{-4phi} gt^ij (R~_ij + R^phi_ij)
//       = e^{-4phi} (gt^ij R~_ij - 8 gt^ij D~_i D~_j phi - 8 gt^ij d_i phi d_j phi)
//   H   = R + 2/3 K^2 - A~_ij A~^ij
//   M_i = Gd^k A~_ik + gt^jk d_j A~_ik + Gamma~^j_jk A~^k_i
//         - Gamma~^k_ji A~^j_k + 6 A~^k_i d_k phi - 2/3 d_i K
//   G^i = Gt^i - gt^jk Gamma~^i_jk
// Norms: every workgroup reduces its points (wave shuffles, then LDS) to 8
// partials; one workgroup then folds the partials in a fixed order, so the
// result does not depend on scheduling.
#include <hip/hip_runtime.h>

#include <mutex>

#include "bssn_api_internal.h"
#include "bssn_kernels.h"
#include "bssn_lds.h"
#include "bssn_stage.h"

namespace bssn {

template <int ORDER, class L>
__device__ __forceinline__ void grad(const L& ld, int s, const double (&ih)[3],
                                     double (&d1)[3]) {
  using F = FD<ORDER>;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double s1 = 0.0;
#pragma unroll
    for (int k = 1; k <= F::M; ++k)
      s1 += F::a(k) * (ld.ax(s, a, k) - ld.ax(s, a, -k));
    d1[a] = s1 * ih[a];
  }
}

// FENCE, here and below: the kernel that reads LDS.  There a compiler fence per
// row of the stencil keeps the row's reads inside the row instead of hoisting all
// of them, which spills registers.  The direct kernels run without: the more
// of their global loads are in flight the better (with the fences a periodic
// 128^3 call takes 923 us at order 4 and 3,580 at order 8, without 599 and
// 2,630).

// Mixed second derivative (the sums of mixed()).
template <int ORDER, bool FENCE, class L>
__device__ __forceinline__ double mixed_rows(const L& ld, int s, int a, int b,
                                             double ihab) {
  using F = FD<ORDER>;
  double acc = 0.0;
#pragma unroll
  for (int i = 1; i <= F::M; ++i) {
    double p = 0.0, m = 0.0;
#pragma unroll
    for (int j = 1; j <= F::M; ++j) {
      p += F::a(j) * (ld.pl(s, a, i, b, j) - ld.pl(s, a, i, b, -j));
      m += F::a(j) * (ld.pl(s, a, -i, b, j) - ld.pl(s, a, -i, b, -j));
    }
    acc += F::a(i) * (p - m);
    if constexpr (FENCE) asm volatile("" : "+v"(acc)::"memory");
  }
  return acc * ihab;
}

// full symmetric Hessian (S-indexed)
template <int ORDER, bool FENCE, class L>
__device__ __forceinline__ void hess(const L& ld, int s, const double (&ih)[3],
                                     double (&dd)[6]) {
  using F = FD<ORDER>;
  const double c0 = ld.c(s);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double s2 = 0.0;
#pragma unroll
    for (int k = 1; k <= F::M; ++k)
      s2 += F::b(k) * ((ld.ax(s, a, k) - c0) + (ld.ax(s, a, -k) - c0));
    if constexpr (FENCE) asm volatile("" : "+v"(s2)::"memory");
    dd[S(a, a)] = s2 * ih[a] * ih[a];
  }
  dd[1] = mixed_rows<ORDER, FENCE>(ld, s, 0, 1, ih[0] * ih[1]);
  dd[2] = mixed_rows<ORDER, FENCE>(ld, s, 0, 2, ih[0] * ih[2]);
  dd[4] = mixed_rows<ORDER, FENCE>(ld, s, 1, 2, ih[1] * ih[2]);
}

// H, M_i and G^i at one point.  The loader's enter(s) opens the phase of slot
// s (in the order of kConSlot); c, ax and pl read it inside its phase, g reads
// gt_ij's centre values at any time.
constexpr int kNCon = 17;
constexpr int kConSlot[kNCon] = {GXX,  GXY,  GXZ, GYY, GYZ, GZZ, GAMX, GAMY,
                                 GAMZ, PHI,  TRK, AXX, AXY, AXZ, AYY,  AYZ,
                                 AZZ};
__host__ __device__ constexpr int con_phase(int s) {
  return s >= GXX && s <= GZZ     ? s - GXX
         : s >= GAMX && s <= GAMZ ? 6 + s - GAMX
         : s == PHI               ? 9
         : s == TRK               ? 10
                                  : 11 + s - AXX;
}

template <int ORDER, bool FENCE, class L>
__device__ __forceinline__ void constraints_point(const L& ld,
                                                  const double (&ih)[3],
                                                  double& H, double (&M)[3],
                                                  double (&Gc)[3]) {
  double gt[6], gu[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) gt[m] = ld.g(GXX + m);
  inverse_metric<double>(gt, gu);
  double dgt[6][3], Rt[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    ld.enter(GXX + m);
    grad<ORDER>(ld, GXX + m, ih, dgt[m]);
    double dd[6];
    hess<ORDER, FENCE>(ld, GXX + m, ih, dd);
    Rt[m] = -0.5 * (gu[0] * dd[0] + gu[3] * dd[3] + gu[5] * dd[5] +
                    2.0 * (gu[1] * dd[1] + gu[2] * dd[2] + gu[4] * dd[4]));
    keep(Rt[m]);
#pragma unroll
    for (int a = 0; a < 3; ++a) keep(dgt[m][a]);
  }
  double Gu[3][6], Gd[3];
  connection<double, FENCE>(dgt, gu, Gu, Gd, Rt);
  double Gt[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double dG[3];
    ld.enter(GAMX + k);
    Gt[k] = ld.c(GAMX + k);
    grad<ORDER>(ld, GAMX + k, ih, dG);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        Rt[S(i, j)] += 0.5 * (gt[S(k, i)] * dG[j] + gt[S(k, j)] * dG[i]);
    // (each phase's sums are finished in it: deferred arithmetic would keep
    // every tap in registers)
#pragma unroll
    for (int m = 0; m < 6; ++m) keep(Rt[m]);
  }
  const double trR = gu[0] * Rt[0] + gu[3] * Rt[3] + gu[5] * Rt[5] +
                     2.0 * (gu[1] * Rt[1] + gu[2] * Rt[2] + gu[4] * Rt[4]);

  double dphi[3], ddphi[6];
  ld.enter(PHI);
  const double phi = ld.c(PHI);
  grad<ORDER>(ld, PHI, ih, dphi);
  hess<ORDER, FENCE>(ld, PHI, ih, ddphi);
  double trDD = 0.0, dphi2 = 0.0;
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const double DD = ddphi[m] - (Gu[0][m] * dphi[0] + Gu[1][m] * dphi[1] +
                                  Gu[2][m] * dphi[2]);
    const double w = (m == 0 || m == 3 || m == 5) ? 1.0 : 2.0;
    trDD += w * gu[m] * DD;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) dphi2 += gu[S(i, j)] * dphi[i] * dphi[j];
  double R = exp(-4.0 * phi) * (trR - 8.0 * trDD - 8.0 * dphi2);
  keep(R);

  ld.enter(TRK);
  const double trK = ld.c(TRK);
  double dK[3];
  grad<ORDER>(ld, TRK, ih, dK);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    M[i] = -(2.0 / 3.0) * dK[i];
    keep(M[i]);
  }
  double At[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    double dA[3];
    ld.enter(AXX + m);
    At[m] = ld.c(AXX + m);
    grad<ORDER>(ld, AXX + m, ih, dA);
    // gt^jk d_j A~_ik: slot m = S(i,k) contributes to M_i and (i != k) M_k
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (S(i, k) == m)
          M[i] += gu[S(0, k)] * dA[0] + gu[S(1, k)] * dA[1] +
                  gu[S(2, k)] * dA[2];
#pragma unroll
    for (int i = 0; i < 3; ++i) keep(M[i]);
  }
  double Aud[3][3], Auu[6];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      Aud[i][j] = gu[S(i, 0)] * At[S(0, j)] + gu[S(i, 1)] * At[S(1, j)] +
                  gu[S(i, 2)] * At[S(2, j)];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i; j < 3; ++j)
      Auu[S(i, j)] = Aud[i][0] * gu[S(0, j)] + Aud[i][1] * gu[S(1, j)] +
                     Aud[i][2] * gu[S(2, j)];
  const double AA = At[0] * Auu[0] + At[3] * Auu[3] + At[5] * Auu[5] +
                    2.0 * (At[1] * Auu[1] + At[2] * Auu[2] + At[4] * Auu[4]);
  H = R + (2.0 / 3.0) * trK * trK - AA;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s += Gd[k] * At[S(i, k)] + 6.0 * Aud[k][i] * dphi[k];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        s += Gu[j][S(j, k)] * Aud[k][i] - Gu[k][S(j, i)] * Aud[j][k];
    }
    M[i] += s;
    const double c = gu[0] * Gu[i][0] + gu[3] * Gu[i][3] + gu[5] * Gu[i][5] +
                     2.0 * (gu[1] * Gu[i][1] + gu[2] * Gu[i][2] +
                            gu[4] * Gu[i][4]);
    Gc[i] = Gt[i] - c;
  }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// partial order: 0 sum H^2, 1 max|H|, 2 sum|M|^2, 3 max|M|, 4 sum|G|^2,
// 5 max|G|, 6 used, 7 non-finite

// The fields of one active point to memory, and its entries of the partials
// (0 at excised points).
__device__ __forceinline__ void point_result(const ConstraintArgs& A, int x,
                                             int y, int z, uint32_t vc,
                                             int32_t nbytes, double H,
                                             const double (&M)[3],
                                             const double (&Gc)[3],
                                             double (&v)[8]) {
  if (A.H) bstore(rsrc(A.H, nbytes), vc, H);
  if (A.M)
#pragma unroll
    for (int i = 0; i < 3; ++i) bstore(rsrc(A.M + i * A.sf, nbytes), vc, M[i]);
  if (A.Gc)
#pragma unroll
    for (int i = 0; i < 3; ++i)
      bstore(rsrc(A.Gc + i * A.sf, nbytes), vc, Gc[i]);
  bool use = true;
  const double xc = A.origin[0] + x * A.h[0], yc = A.origin[1] + y * A.h[1],
               zc = A.origin[2] + z * A.h[2];
  for (int c = 0; c < A.ncent; ++c) {
    const double dx = xc - A.centres[c][0], dy = yc - A.centres[c][1],
                 dz = zc - A.centres[c][2];
    if (sqrt(dx * dx + dy * dy + dz * dz) <= A.r_exc) use = false;
  }
  const double m2 = M[0] * M[0] + M[1] * M[1] + M[2] * M[2];
  const double g2 = Gc[0] * Gc[0] + Gc[1] * Gc[1] + Gc[2] * Gc[2];
  const double mm = sqrt(m2), gm = sqrt(g2);
  const bool fin = isfinite(H) && isfinite(mm) && isfinite(gm);
  const bool in = use && fin;
  v[0] = in ? H * H : 0.0;
  v[1] = in ? fabs(H) : 0.0;
  v[2] = in ? mm * mm : 0.0;
  v[3] = in ? mm : 0.0;
  v[4] = in ? gm * gm : 0.0;
  v[5] = in ? gm : 0.0;
  v[6] = in ? 1.0 : 0.0;
  v[7] = use && !fin ? 1.0 : 0.0;
}

// The workgroup's partials (4 waves) to out[0..7].
__device__ __forceinline__ void block_partials(const double (&v)[8], int tid,
                                               double (*red)[4], double* out) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const bool mx = (k == 1 || k == 3 || k == 5);
    const double w = mx ? wave_max(v[k]) : wave_sum(v[k]);
    if ((tid & 63) == 0) red[k][tid >> 6] = w;
  }
  __syncthreads();
  if (tid < 8) {
    const bool mx = (tid == 1 || tid == 3 || tid == 5);
    double acc = red[tid][0];
    for (int w = 1; w < 4; ++w)
      acc = mx ? fmax(acc, red[tid][w]) : acc + red[tid][w];
    out[tid] = acc;
  }
}

template <int ORDER, bool PERIODIC>
__global__ void __launch_bounds__(256)
    k_constraints(const ConstraintArgs A, double* __restrict__ partials) {
  constexpr int R = FD<ORDER>::R;
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  const bool active = x < A.n[0] && y < A.n[1];
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (active) {
    const int g = A.ghost;
    const int32_t nbytes = int32_t(A.sf * 8);
    const uint32_t sy8 = uint32_t(A.sy) * 8u, sz8 = uint32_t(A.sz) * 8u;
    const uint32_t vc =
        uint32_t(z + g) * sz8 + uint32_t(y + g) * sy8 + uint32_t(x + g) * 8u;
    const double ih[3] = {1.0 / A.h[0], 1.0 / A.h[1], 1.0 / A.h[2]};
    double H, M[3], Gc[3];
    if constexpr (!PERIODIC) {
      LdStatic<R> ld;
      ld.u = A.u;
      ld.sf = A.sf;
      ld.nbytes = nbytes;
      ld.vlo = vc - uint32_t(R) * (8u + sy8 + sz8);
      ld.str[0] = 8u;
      ld.str[1] = sy8;
      ld.str[2] = sz8;
      constraints_point<ORDER, false>(ld, ih, H, M, Gc);
    } else {
      LdPeriodic<R> ld;
      ld.u = A.u;
      ld.sf = A.sf;
      ld.nbytes = nbytes;
      const int pos[3] = {x, y, z};
      const uint32_t st[3] = {8u, sy8, sz8};
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int k = -R; k <= R; ++k) {
          int q = pos[a] + k;
          q = q < 0 ? q + A.n[a] : (q >= A.n[a] ? q - A.n[a] : q);
          ld.o[a][R + k] = uint32_t(q + g) * st[a];
        }
      constraints_point<ORDER, false>(ld, ih, H, M, Gc);
    }
    point_result(A, x, y, z, vc, nbytes, H, M, Gc, v);
  }
  __shared__ double red[8][4];
  const size_t b =
      blockIdx.x + gridDim.x * (blockIdx.y + size_t(gridDim.y) * blockIdx.z);
  block_partials(v, threadIdx.x + threadIdx.y * blockDim.x, red,
                    partials + b * 8);
}

// ---- static grids: boxes staged in LDS -----------------------------------------
// One workgroup of 256 threads per 16 x 4 x 4 tile, one point per thread, two
// workgroups per CU.  The haloed box of each slot, (16 + 2M) x (4 + 2M) x
// (4 + 2M) doubles (M: reach of the centred stencils), is moved into one of NB
// LDS buffers by buffer->LDS DMA, NB - 1 phases ahead.  What bounded the
// direct kernel was its 500 to 1,500 global loads per point; here a tap is an
// LDS read and each box is fetched once per tile.  A 128^3 call with fields and
// norms takes 331 us at order 4 (it moves 403 MB, so 1.2 TB/s), 604 in the
// direct kernel; what is left is the latency of the LDS reads and the algebra
// at two waves per SIMD.
template <int ORDER>
struct ConGeo {
  static constexpr int M = FD<ORDER>::M, TX = kLdsTile[0], TY = kLdsTile[1],
                       TZ = kLdsTile[2];
  static constexpr int W = TX + 2 * M, H = TY + 2 * M, D = TZ + 2 * M;
  static constexpr int G = W * H * D / 2, NI = (G + 63) / 64,
                       L = (NI + 3) / 4, BUFD = NI * 128;
  static constexpr int NB = ORDER == 4 ? 6 : 2;
  static constexpr int CL = 3;  // centre block: 6 slots, 3 instructions a wave
};

template <int ORDER>
struct ConLds {
  double box[ConGeo<ORDER>::NB][ConGeo<ORDER>::BUFD];
  double cen[6 * 256];
  double red[8][4];
};

template <int ORDER>
struct LdCon {
  using Geo = ConGeo<ORDER>;
  const ConstraintArgs& A;
  ConLds<ORDER>& S;
  const int wave, lane;
  const uint32_t tb;
  uint32_t off[Geo::L];
  mutable const lds_double* pc;

  __device__ __forceinline__ void issue(int p) const {
    const v4i d = slot_dma_rsrc(A.u, A.sf, kConSlot[p], int32_t(A.sf * 8));
    const uint32_t l0 = lds_addr(S.box[p % Geo::NB]) +
                        uint32_t(wave * Geo::L) * 1024u;
#pragma unroll
    for (int j = 0; j < Geo::L; ++j)
      if (j < Geo::NI - 3 * Geo::L || wave < 3)
        dma16(d, off[j] + tb, l0 + j * 1024u);
  }
  // boxes issued after phase p's when it is waited for, in instructions
  template <int P, int PER_BOX>
  __device__ __forceinline__ void wait() const {
    constexpr int later =
        P + Geo::NB - 2 < kNCon - 1 ? Geo::NB - 2 : kNCon - 1 - P;
    vm_wait_n<later * PER_BOX>();
  }
  template <int P>
  __device__ __forceinline__ void open() const {
    if (wave < 3)
      wait<P, Geo::L>();
    else
      wait<P, Geo::NI - 3 * Geo::L>();
    __builtin_amdgcn_s_barrier();
    // the buffer of phase P - 1 is free
    if constexpr (P + Geo::NB - 1 < kNCon) issue(P + Geo::NB - 1);
    const int tx = lane & 15, ty = lane >> 4;
    const lds_double* b = (const lds_double*)S.box[P % Geo::NB] +
                          (wave * Geo::H + ty) * Geo::W + tx;
    asm volatile("" : "+v"(b));
    pc = b;
  }
  __device__ __forceinline__ void enter(int s) const {
    switch (con_phase(s)) {
      case 0: return open<0>();
      case 1: return open<1>();
      case 2: return open<2>();
      case 3: return open<3>();
      case 4: return open<4>();
      case 5: return open<5>();
      case 6: return open<6>();
      case 7: return open<7>();
      case 8: return open<8>();
      case 9: return open<9>();
      case 10: return open<10>();
      case 11: return open<11>();
      case 12: return open<12>();
      case 13: return open<13>();
      case 14: return open<14>();
      case 15: return open<15>();
      case 16: return open<16>();
    }
  }
  __device__ __forceinline__ double g(int s) const {
    return ((const lds_double*)S.cen)[(s - GXX) * 256 + wave * 64 + lane];
  }
  static constexpr int kC = Geo::M * (1 + Geo::W + Geo::W * Geo::H);
  __device__ __forceinline__ static constexpr int str(int a) {
    return a == 0 ? 1 : (a == 1 ? Geo::W : Geo::W * Geo::H);
  }
  __device__ __forceinline__ double c(int) const { return pc[kC]; }
  __device__ __forceinline__ double ax(int, int a, int k) const {
    return pc[kC + k * str(a)];
  }
  __device__ __forceinline__ double pl(int, int a, int i, int b, int j) const {
    return pc[kC + i * str(a) + j * str(b)];
  }
};

template <int ORDER>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_constraints_lds(const ConstraintArgs A, const int ntx, const int nty,
                      const int ntile, double* __restrict__ partials) {
  using Geo = ConGeo<ORDER>;
  __shared__ __attribute__((aligned(16))) ConLds<ORDER> L;
  // the XCD (block id mod 8) takes a contiguous eighth of the tiles (x
  // fastest), so neighbouring tiles share an L2
  const int per = (ntile + 7) / 8;
  const int tile = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
  if (int(blockIdx.x >> 3) >= per || tile >= ntile) return;
  const int x0 = tile % ntx * Geo::TX, y0 = tile / ntx % nty * Geo::TY,
            z0 = tile / (ntx * nty) * Geo::TZ;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = A.ghost;
  const int32_t nbytes = int32_t(A.sf * 8);
  const uint32_t sy8 = uint32_t(A.sy) * 8u, sz8 = uint32_t(A.sz) * 8u;
  LdCon<ORDER> ld{A, L, wave, lane,
                  uint32_t(z0 + g - Geo::M) * sz8 +
                      uint32_t(y0 + g - Geo::M) * sy8 +
                      uint32_t(x0 + g - Geo::M) * 8u};
#pragma unroll
  for (int j = 0; j < Geo::L; ++j) {
    const int i = (wave * Geo::L + j) * 64 + lane;
    const int col = i % (Geo::W / 2), row = i / (Geo::W / 2);
    ld.off[j] = i < Geo::G ? uint32_t(row / Geo::H) * sz8 +
                                 uint32_t(row % Geo::H) * sy8 + col * 16u
                           : 0x80000000u;
  }
  // the metric at the tile's points: instruction j of wave w moves half of
  // slot GXX + (3 w + j) / 2
#pragma unroll
  for (int j = 0; j < Geo::CL; ++j) {
    const int ins = wave * Geo::CL + j;
    const int row = (ins & 1) * 8 + (lane >> 3);
    const uint32_t o = uint32_t(z0 + (row >> 2) + g) * sz8 +
                       uint32_t(y0 + (row & 3) + g) * sy8 +
                       uint32_t(x0 + g + 2 * (lane & 7)) * 8u;
    dma16(slot_dma_rsrc(A.u, A.sf, GXX + (ins >> 1), nbytes), o,
          lds_addr(L.cen) + uint32_t(ins) * 1024u);
  }
#pragma unroll
  for (int p = 0; p < Geo::NB - 1; ++p) ld.issue(p);
  const int x = x0 + (lane & 15), y = y0 + (lane >> 4), z = z0 + wave;
  const double ih[3] = {1.0 / A.h[0], 1.0 / A.h[1], 1.0 / A.h[2]};
  // the centre block is older than the boxes still in flight here
  if (wave < 3)
    vm_wait_n<(Geo::NB - 1) * Geo::L>();
  else
    vm_wait_n<(Geo::NB - 1) * (Geo::NI - 3 * Geo::L)>();
  __builtin_amdgcn_s_barrier();
  double H, M[3], Gc[3];
  constraints_point<ORDER, true>(ld, ih, H, M, Gc);
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (x < A.n[0] && y < A.n[1] && z < A.n[2]) {
    const uint32_t vc =
        uint32_t(z + g) * sz8 + uint32_t(y + g) * sy8 + uint32_t(x + g) * 8u;
    point_result(A, x, y, z, vc, nbytes, H, M, Gc, v);
  }
  block_partials(v, tid, L.red, partials + size_t(tile) * 8);
}

// One workgroup folds nb partial records in a fixed order: thread t takes value
// t mod 8 of the records t / 8, t / 8 + 128, ..., so a wave reads 512 contiguous
// bytes (a whole record per thread touched 64 lines per load and took 18 us for
// 8,192 records; this takes 14).
__global__ void __launch_bounds__(1024)
    k_norms(const double* __restrict__ partials, long nb,
            double* __restrict__ norms) {
  __shared__ double red[8][16], tot[8];
  const int t = threadIdx.x, k = t & 7;
  const bool mx = (k == 1 || k == 3 || k == 5);
  double v = 0;
#pragma unroll 8
  for (long b = t >> 3; b < nb; b += 128) {
    const double p = partials[b * 8 + k];
    v = mx ? fmax(v, p) : v + p;
  }
#pragma unroll
  for (int off = 32; off >= 8; off >>= 1) {
    const double w = __shfl_xor(v, off, 64);
    v = mx ? fmax(v, w) : v + w;
  }
  if ((t & 63) < 8) red[k][t >> 6] = v;
  __syncthreads();
  if (t < 8) {
    double acc = red[t][0];
    for (int w = 1; w < 16; ++w)
      acc = mx ? fmax(acc, red[t][w]) : acc + red[t][w];
    tot[t] = acc;
  }
  __syncthreads();
  if (t == 0) {
    const double n = tot[6];
    norms[0] = n > 0 ? sqrt(tot[0] / n) : 0.0;
    norms[1] = tot[1];
    norms[2] = n > 0 ? sqrt(tot[2] / n) : 0.0;
    norms[3] = tot[3];
    norms[4] = n > 0 ? sqrt(tot[4] / n) : 0.0;
    norms[5] = tot[5];
    norms[6] = n;
    norms[7] = tot[7];
  }
}

static void cgrid(const ConstraintArgs& A, dim3& grd, dim3& blk) {
  const int bx = A.n[0] > 32 ? 64 : 32;
  blk = dim3(bx, 256 / bx, 1);
  grd = dim3((A.n[0] + bx - 1) / bx, (A.n[1] + blk.y - 1) / blk.y, A.n[2]);
}

int constraint_blocks(const ConstraintArgs& A) {
  dim3 g, b;
  cgrid(A, g, b);
  return int(g.x * g.y * g.z);
}

hipError_t launch_constraints(const ConstraintArgs& A, int order,
                              double* partials, int nblocks_max,
                              double* norms, hipStream_t st) {
  dim3 grd, blk;
  cgrid(A, grd, blk);
  const long nb = long(grd.x) * grd.y * grd.z;
  if (nb > nblocks_max) return hipErrorInvalidValue;
  const int ntx = (A.n[0] + kLdsTile[0] - 1) / kLdsTile[0],
            nty = (A.n[1] + kLdsTile[1] - 1) / kLdsTile[1],
            ntz = (A.n[2] + kLdsTile[2] - 1) / kLdsTile[2];
  const long ntile = long(ntx) * nty * ntz;
  // The LDS kernel takes static grids whose rows allow 16-byte granules and
  // that have no more tiles than the direct kernel has workgroups (grids thin
  // in z do), so that both need the same workspace.
  if (!A.periodic && ntile <= nb &&
      (reinterpret_cast<uintptr_t>(A.u) + 8u * uintptr_t(A.ghost)) % 16 == 0 &&
      A.sy % 2 == 0 && A.sz % 2 == 0 && A.sf % 2 == 0) {
    const dim3 g(unsigned(8 * ((ntile + 7) / 8)));
    if (order == 4)
      hipLaunchKernelGGL(k_constraints_lds<4>, g, dim3(256), 0, st, A, ntx,
                         nty, int(ntile), partials);
    else
      hipLaunchKernelGGL(k_constraints_lds<8>, g, dim3(256), 0, st, A, ntx,
                         nty, int(ntile), partials);
    hipLaunchKernelGGL(k_norms, dim3(1), dim3(1024), 0, st, partials, ntile,
                       norms);
    return hipGetLastError();
  }
  if (order == 4) {
    if (A.periodic)
      hipLaunchKernelGGL((k_constraints<4, true>), grd, blk, 0, st, A, partials);
    else
      hipLaunchKernelGGL((k_constraints<4, false>), grd, blk, 0, st, A, partials);
  } else {
    if (A.periodic)
      hipLaunchKernelGGL((k_constraints<8, true>), grd, blk, 0, st, A, partials);
    else
      hipLaunchKernelGGL((k_constraints<8, false>), grd, blk, 0, st, A, partials);
  }
  hipLaunchKernelGGL(k_norms, dim3(1), dim3(1024), 0, st, partials, nb, norms);
  return hipGetLastError();
}

// ---- mixed-precision routing statistics ----------------------------------------
__global__ void __launch_bounds__(256)
    k_tile_count(const Patch P, const double thr,
                 unsigned long long* __restrict__ counter) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  const bool active = x < P.n[0] && y < P.n[1];
  const int g = P.ghost;
  const uint32_t vc = uint32_t(z + g) * uint32_t(P.sz) * 8u +
                      uint32_t(y + g) * uint32_t(P.sy) * 8u +
                      uint32_t(x + g) * 8u;
  const bool f64 = tile_needs_fp64(P, active, vc, int32_t(P.sf * 8), thr);
  if (threadIdx.x == 0 && threadIdx.y == 0 && f64) atomicAdd(counter, 1ull);
}

// The same predicate over the LDS kernel's 16 x 4 x 4 tiles (one block per
// tile, thread = point as in that kernel).
__global__ void __launch_bounds__(256)
    k_tile_count_lds(const Patch P, const double thr, const int ntx,
                     const int nty, unsigned long long* __restrict__ counter) {
  const int t = blockIdx.x, tid = threadIdx.x;
  const int ix = t % ntx, iy = (t / ntx) % nty, iz = t / (ntx * nty);
  const int x = ix * kLdsTile[0] + (tid & 15);
  const int y = iy * kLdsTile[1] + ((tid >> 4) & 3);
  const int z = iz * kLdsTile[2] + (tid >> 6);
  const bool active = x < P.n[0] && y < P.n[1] && z < P.n[2];
  const int g = P.ghost;
  const uint32_t vc = uint32_t(z + g) * uint32_t(P.sz) * 8u +
                      uint32_t(y + g) * uint32_t(P.sy) * 8u +
                      uint32_t(x + g) * 8u;
  const bool f64 = tile_needs_fp64(P, active, vc, int32_t(P.sf * 8), thr);
  if (tid == 0 && f64) atomicAdd(counter, 1ull);
}

void tile_grid(const Patch& P, int lds, dim3& grd, dim3& blk) {
  if (lds) {
    const int ntx = (P.n[0] + kLdsTile[0] - 1) / kLdsTile[0];
    const int nty = (P.n[1] + kLdsTile[1] - 1) / kLdsTile[1];
    const int ntz = (P.n[2] + kLdsTile[2] - 1) / kLdsTile[2];
    grd = dim3(ntx * nty * ntz, 1, 1);
    blk = dim3(256, 1, 1);
    return;
  }
  stage_tile_shape(P, 0, blk);
  grd = dim3((P.n[0] + blk.x - 1) / blk.x, (P.n[1] + blk.y - 1) / blk.y,
             P.n[2]);
}

hipError_t launch_tile_count(const Patch& P, double thr, int lds,
                             unsigned long long* counter, hipStream_t st) {
  dim3 grd, blk;
  tile_grid(P, lds, grd, blk);
  if (lds) {
    const int ntx = (P.n[0] + kLdsTile[0] - 1) / kLdsTile[0];
    const int nty = (P.n[1] + kLdsTile[1] - 1) / kLdsTile[1];
    hipLaunchKernelGGL(k_tile_count_lds, grd, blk, 0, st, P, thr, ntx, nty,
                       counter);
  } else {
    hipLaunchKernelGGL(k_tile_count, grd, blk, 0, st, P, thr, counter);
  }
  return hipGetLastError();
}

}  // namespace bssn

// ---- constraints without allocation ---------------------------------------------
// The per-block partial norms of bssn_constraints_noalloc live in this
// file-scope device array: kNoAllocRecords records of 8 doubles (16 MiB),
// which covers grids of up to 262,144 constraint blocks (a 384^3 grid needs
// 221,184).  Each GPU holds its own copy for the life of the process.  Host
// code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): it uses the device address that
// hipGetSymbolAddress returns, once per device, with that device current.
namespace bssn {
constexpr int kNoAllocRecords = 1 << 18;
static __device__ __align__(256) double scratch[size_t(kNoAllocRecords) * 8];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of `scratch` (set up on the first
// call on the device).
int scratch_address(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices)
    return fail(BSSN_EUNSUPPORTED, "device %d beyond the %d the library "
                "tracks", dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return BSSN_OK;
}
}  // namespace
}  // namespace bssn

extern "C" int bssn_constraints_noalloc(const bssn_grid* grid,
                                        const bssn_params* params,
                                        const double* u, double* H,
                                        double* M, double* G,
                                        const double* centres, int ncent,
                                        double r_exc, double* norms,
                                        void* stream) {
  using namespace bssn;
  ConstraintArgs A{};
  int rc = constraint_args(grid, params, u, H, M, G, centres, ncent, r_exc,
                           norms, &A);
  if (rc) return rc;
  const long nb = constraint_blocks(A);
  if (nb > kNoAllocRecords)
    return fail(BSSN_EINVAL, "the grid needs %ld partial records; the "
                "allocation-free constraints hold at most %d (a 384^3 grid "
                "needs 221184)", nb, kNoAllocRecords);
  double* part = nullptr;
  if ((rc = scratch_address(&part))) return rc;
  // every record a launch reads is written by the same launch: nothing to
  // clear
  const hipError_t e = launch_constraints(A, params->fd_order, part,
                                          kNoAllocRecords, norms,
                                          (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "bssn_constraints_noalloc launch");
  return BSSN_OK;
}
