// bssn_split.h -- the fused RHS + RK4 stage with two waves per 64 points.
//
// A workgroup of 512 threads owns one 16 x 4 x 4 tile at a time.  Each point
// belongs to two threads, whose registers (256 each) share its working set:
//   * the curvature waves (0..3, wave w = plane w of the tile) form the
//     derivatives and the pointwise algebra, and issue the buffer->LDS DMA of
//     the stencil boxes;
//   * the transport waves (4..7) form the advection + dissipation sum of
//     every slot and run the RK4 update: the loads and stores of u_n, acc and
//     the stage output.
// One wave per SIMD (a whole point per thread needs more than 256 registers)
// leaves the issue slots of every LDS round trip, dependent FP64 result and
// memory wait empty; the second wave fills them.
//
// The 25 slots stream through LDS in 11 steps.  A step holds one "heavy"
// slot (one with mixed second derivatives: gt_ij, phi, alpha, beta^i), as a
// haloed box of (16 + 2R + 1) x (4 + 2R) x (4 + 2R) doubles, and one or two
// "light" slots (A~_ij, Gt^i, K, B^i, A), whose stencils only read the three
// axis lines through each point and which are stored as three runs: the
// tile's rows extended in x, its columns extended in y, and in z (a third of
// a box at order 4, 0.4 at order 8).  While step s is worked on, the DMA of
// step s + 1 fills the other buffers; one barrier separates the steps.
//
// Mixed second derivatives: the inner first-difference sums are formed once
// per position by all eight waves (MixGeo), shared through LDS, and read
// back by the curvature waves after a second barrier.
//
// The curvature waves hand 17 sums per point to the transport waves through
// LDS at the end of a tile.  The transport waves apply the RK4 update of a
// tile during the next one, at each step for the slots of that step (whose
// registers that step then reuses), so that its loads and stores are spread
// over the whole tile time instead of meeting in one burst.
//
// What bounds it: the two waves of a SIMD are close to balanced and both
// latency-bound (an order-4 tile takes about 41,000 cycles: the SIMDs issue
// vector instructions in 46% of them and scalar ones in 22%, the LDS is busy in
// 43%, a wave spends 39% in waits and barriers); the DMA takes about 15,000
// cycles of the CU's address unit, and its issue blocks the wave
// for 100-150 cycles per instruction, so it sits in the curvature waves,
// whose arithmetic is the shorter, right after the barrier that the inner
// sums need anyway.  Measured against one wave per SIMD with the whole point
// in each thread (RK4 step, one MI355X): 128^3 order 4 2.91 -> 2.45 ms, 256^3
// order 4 25.4 -> 19.7 ms, 256^3 order 8 36.4 -> 28.6 ms, 83 x 61 x 45 order 4
// 531 -> 376 us, 48 uneven patches 18.7 -> 17.1 ms (14.8 with dealt tiles); FP32 at order 8 (mixed
// precision, 97 x 53 x 75) 1,463 -> 1,076 us.  Prefetching one step ahead
// instead of two (order 4) cost 8%, updating at the start of a step instead of
// its end 10%; a branch around the update's loads or stores costs 10-80%, as
// the compiler then waits for the loads at the branch.
#pragma once
#include <hip/hip_runtime.h>

#include "bssn_lds.h"

namespace bssn {

constexpr int kNStep = 11;
constexpr int kStepHeavy[kNStep] = {GXX, GXY, GXZ, GYY,  GYZ, GZZ,
                                    PHI, ALP, BETX, BETY, BETZ};
// the light slots of step s: kStepLight[kStepLight0[s] .. kStepLight0[s+1])
// and, at order 8, the light buffer (of three) each uses; neighbouring steps
// (cyclically) never share one
// (the steps with the longest algebra, 5 and 10, have two)
constexpr int kStepLight0[kNStep + 1] = {0, 1, 2, 4, 5, 6, 8, 9, 10, 11, 12,
                                         14};
constexpr int kStepLight[14] = {AXX,  AXY,  AXZ, GAMX, AYY, AYZ, AZZ,
                                GAMY, GAMZ, TRK, BX,   BY,  BZ,  ADOT};
constexpr int kLightBuf[14] = {2, 0, 1, 2, 0, 1, 0, 2, 1, 0, 1, 2, 0, 1};
__host__ __device__ constexpr int n_light(int s) { return kStepLight0[s + 1] - kStepLight0[s]; }
// the i-th slot of step s: its heavy slot, then its light ones
__host__ __device__ constexpr int step_slot(int s, int i) {
  return i == 0 ? kStepHeavy[s] : kStepLight[kStepLight0[s] + i - 1];
}

template <int ORDER>
struct SplitGeo {
  static constexpr int R = FD<ORDER>::R, MX = FD<ORDER>::M;
  static constexpr int TX = kLdsTile[0], TY = kLdsTile[1], TZ = kLdsTile[2];
  static constexpr int W = (TX + 2 * R + 3) / 2 * 2;  // even, one pad column
  static constexpr int H = TY + 2 * R, D = TZ + 2 * R;
  // heavy box: G granules of 16 bytes, NI DMA instructions of 64 lanes, at
  // most L per curvature wave
  static constexpr int G = W * H * D / 2, NI = (G + 63) / 64,
                       L = (NI + 3) / 4, BUFD = NI * 128;
  // light slot: x, y and z runs
  static constexpr int LX = TZ * TY * W, LY = TZ * H * TX, LZ = D * TY * TX;
  static constexpr int LG = (LX + LY + LZ) / 2, LNI = (LG + 63) / 64,
                       LL = (LNI + 3) / 4, LBUFD = LNI * 128;
  // the handed-over sums lie in the heavy buffer of the tile's last step
  // (order 8, where LDS is full) or in an array of their own
  static constexpr bool HAND_IN_BOX = ORDER == 8;
  // Prefetch.  Order 4 has LDS for three heavy and four light buffers: the
  // slots of step s + 2 are fetched during step s.  Order 8 has two and
  // three: the heavy slot of step s + 2 is fetched into the box of step s
  // once every wave has read that (LATE: a barrier after the heavy slot's
  // stencils), the light ones of step s + 1 during step s.
  static constexpr bool LATE = ORDER == 8;
  static constexpr int NH = LATE ? 2 : 3, NLB = LATE ? 3 : 4;
  // buffer of the heavy slot of step s of a workgroup's k-th tile, and of
  // the light entry i (any window of three steps holds at most four)
  __device__ static __forceinline__ int heavy_buf(int k, int s) {
    return LATE ? (k + s) & 1 : unsigned(2 * k + s) % 3u;
  }
  __device__ static __forceinline__ int light_buf(int k, int i) {
    return LATE ? kLightBuf[i] : (2 * k + i) & 3;
  }
};
constexpr int kNHand = 17;  // gt_ij, A~_ij, Gt^i, K, phi

// the handed-over sums' own array, where they have one
template <typename T, bool IN_BOX>
struct HandLds {
  T hand[kNHand * 256];
};
template <typename T>
struct HandLds<T, true> {
  static constexpr T* hand = nullptr;
};
template <int ORDER, typename T>
struct SplitLds : HandLds<T, SplitGeo<ORDER>::HAND_IN_BOX> {
  using Geo = SplitGeo<ORDER>;
  double heavy[Geo::NH * Geo::BUFD];
  double light[Geo::NLB * Geo::LBUFD];
  double cen[4 * 256];  // beta^i and alpha at the tile's points
  T mix[MixGeo<Geo>::NE];
};

// The barrier inside a step: this wave's LDS accesses have completed.
__device__ __forceinline__ void mid_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// The barrier between steps in a curvature wave: all of its DMA but the N
// youngest instructions has landed too.
template <int N>
__device__ __forceinline__ void step_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N)
               : "memory");
}

// ---- stencils on the LDS layouts -----------------------------------------------
// Taps of a point in a heavy box, from its stencil corner (x-R, y-R, z-R).
template <int ORDER>
struct HeavyTaps {
  using Geo = SplitGeo<ORDER>;
  const lds_double* p;
  static constexpr int kC = Geo::R * (1 + Geo::W + Geo::W * Geo::H);
  __device__ __forceinline__ HeavyTaps(const lds_double* q) : p(q) {
    asm volatile("" : "+v"(p));
  }
  __device__ __forceinline__ double c() const { return p[kC]; }
  __device__ __forceinline__ double ax(int a, int k) const {
    return p[kC + k * (a == 0 ? 1 : (a == 1 ? Geo::W : Geo::W * Geo::H))];
  }
};
// Taps of a point in the three runs of a light slot, from the lowest of each.
template <int ORDER>
struct LightTaps {
  using Geo = SplitGeo<ORDER>;
  const lds_double *x, *y, *z;
  __device__ __forceinline__ LightTaps(const lds_double* q, int ox, int oy,
                                       int oz)
      : x(q + ox), y(q + oy), z(q + oz) {
    asm volatile("" : "+v"(x), "+v"(y), "+v"(z));
  }
  __device__ __forceinline__ double c() const { return x[Geo::R]; }
  __device__ __forceinline__ double ax(int a, int k) const {
    return a == 0   ? x[Geo::R + k]
           : a == 1 ? y[(Geo::R + k) * Geo::TX]
                    : z[(Geo::R + k) * Geo::TX * Geo::TY];
  }
};
// Offsets of the lowest taps of the point (lane, plane w) in a light buffer.
template <int ORDER>
struct LightOffsets {
  using Geo = SplitGeo<ORDER>;
  int x, y, z;
  __device__ __forceinline__ LightOffsets(int w, int lane) {
    const int tx = lane & 15, ty = lane >> 4;
    x = (w * Geo::TY + ty) * Geo::W + tx + 1;
    y = Geo::LX + (w * Geo::H + ty) * Geo::TX + tx;
    z = Geo::LX + Geo::LY + w * Geo::TX * Geo::TY + lane;
  }
};

// Advection + dissipation sum of one slot (the taps of the next axis are
// read before this axis's arithmetic, two FMA chains per axis).
template <int ORDER, typename T, class TP>
__device__ __forceinline__ T drift(const TP& t,
                                   const T (&cw)[3][2 * FD<ORDER>::R]) {
  constexpr int R = FD<ORDER>::R;
  const double c0 = t.c();
  T adv = T(0);
  double u[2][2 * R];
#pragma unroll
  for (int k = -R; k <= R; ++k)
    if (k != 0) u[0][WI<R>(k)] = t.ax(0, k);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (a < 2) {
#pragma unroll
      for (int k = -R; k <= R; ++k)
        if (k != 0) u[(a + 1) & 1][WI<R>(k)] = t.ax(a + 1, k);
    }
    T lo = T(0), hi = T(0);
#pragma unroll
    for (int k = 1; k <= R; ++k) {
      lo += cw[a][WI<R>(-k)] * T(u[a & 1][WI<R>(-k)] - c0);
      hi += cw[a][WI<R>(k)] * T(u[a & 1][WI<R>(k)] - c0);
    }
    adv += lo + hi;
    keep(adv);
  }
  return adv;
}

// First and (D2) pure second derivatives of one slot.
template <int ORDER, typename T, bool D2, class TP>
__device__ __forceinline__ void derivs(const TP& t, const T (&ih)[3],
                                       const T (&ih2)[3], T (&d1)[3],
                                       T (&d2)[3]) {
  using F = FD<ORDER>;
  constexpr int M = F::M;
  const double c0 = D2 ? t.c() : 0.0;
  double u[2][2 * M];
#pragma unroll
  for (int k = 1; k <= M; ++k) {
    u[0][2 * k - 2] = t.ax(0, k);
    u[0][2 * k - 1] = t.ax(0, -k);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (a < 2) {
#pragma unroll
      for (int k = 1; k <= M; ++k) {
        u[(a + 1) & 1][2 * k - 2] = t.ax(a + 1, k);
        u[(a + 1) & 1][2 * k - 1] = t.ax(a + 1, -k);
      }
    }
    T s1 = T(0), s2 = T(0);
#pragma unroll
    for (int k = 1; k <= M; ++k) {
      const double p = u[a & 1][2 * k - 2], m = u[a & 1][2 * k - 1];
      s1 += T(F::a(k)) * T(p - m);
      if constexpr (D2) s2 += T(F::b(k)) * T((p - c0) + (m - c0));
    }
    d1[a] = s1 * ih[a];
    keep(d1[a]);
    if constexpr (D2) {
      d2[a] = s2 * ih2[a];
      keep(d2[a]);
    }
  }
}

// ---- shared inner sums of the mixed second derivatives ------------------------
// One inner sum per lane: entry `e` is the element of its lowest tap, S the
// tap stride (W: y sums, W H: z sums).
template <int ORDER, int S>
struct InnerSum {
  static constexpr int M = FD<ORDER>::M;
  double t[2 * M];
  __device__ __forceinline__ void read(const lds_double* b) {
    asm("" : "+v"(b));
#pragma unroll
    for (int j = 1; j <= M; ++j) {
      t[2 * j - 2] = b[(M + j) * S];
      t[2 * j - 1] = b[(M - j) * S];
    }
  }
  template <typename T>
  __device__ __forceinline__ T sum() const {
    T v = T(0);
#pragma unroll
    for (int j = 1; j <= M; ++j)
      v += T(FD<ORDER>::a(j)) * T(t[2 * j - 2] - t[2 * j - 1]);
    return v;
  }
};

// The chunks of MixGeo (64 entries each: PX y sums, QX z sums, PZ y sums) of
// one wave of either kind.  Chunk ranges, w = 0..3:
//   order 8: curvature PZ 12 + w, PZ 16 + w, PX 0 + w;
//            transport PX 4, 5 and QX 6, 7 (w = 0..3), QX 8 + w;
//   order 4: curvature PZ 10 + w;
//            transport PX 0 + w, QX 5 + w, then PX 4 (w = 2), QX 9 (w = 3).
template <int ORDER, typename T, bool TRANSPORT>
__device__ __forceinline__ void inner_sums(const lds_double* box, T* mix_,
                                           int w, int lane) {
  using Geo = SplitGeo<ORDER>;
  using MG = MixGeo<Geo>;
  constexpr int SY = Geo::W, SZ = Geo::W * Geo::H;
  static_assert(MG::NC == (ORDER == 8 ? 20 : 14), "chunk ranges");
  typedef __attribute__((address_space(3))) T lds_t;
  lds_t* mix = (lds_t*)mix_ + lane;
  // the lane number through an opaque copy: entry positions are formed here
  // rather than held in registers through the tile loop
  int ln = lane;
  asm volatile("" : "+v"(ln));
  auto entry = [&](int c) { return box + mix_entry<Geo>(c, ln); };
  if constexpr (!TRANSPORT && ORDER == 8) {
    InnerSum<8, SY> a, b, c;
    a.read(entry(12 + w));
    b.read(entry(16 + w));
    mix[(12 + w) * 64] = a.template sum<T>();
    c.read(entry(w));
    mix[(16 + w) * 64] = b.template sum<T>();
    mix[w * 64] = c.template sum<T>();
  } else if constexpr (!TRANSPORT) {
    InnerSum<4, SY> a;
    a.read(entry(10 + w));
    mix[(10 + w) * 64] = a.template sum<T>();
  } else if constexpr (ORDER == 8) {
    InnerSum<8, SZ> b;
    b.read(entry(8 + w));
    if (w < 2) {
      path_mark<0>();
      InnerSum<8, SY> a;
      a.read(entry(4 + w));
      mix[(4 + w) * 64] = a.template sum<T>();
      path_mark<0>();
    } else {
      path_mark<1>();
      InnerSum<8, SZ> a;
      a.read(entry(4 + w));
      mix[(4 + w) * 64] = a.template sum<T>();
      path_mark<1>();
    }
    mix[(8 + w) * 64] = b.template sum<T>();
  } else {
    InnerSum<4, SY> a;
    InnerSum<4, SZ> b;
    a.read(entry(w));
    b.read(entry(5 + w));
    mix[w * 64] = a.template sum<T>();
    mix[(5 + w) * 64] = b.template sum<T>();
    if (w == 2) {
      path_mark<0>();
      a.read(entry(4));
      mix[4 * 64] = a.template sum<T>();
      path_mark<0>();
    } else if (w == 3) {
      path_mark<1>();
      b.read(entry(9));
      mix[9 * 64] = b.template sum<T>();
      path_mark<1>();
    }
  }
}

// d_x d_y, d_x d_z, d_y d_z of the step's heavy slot at the point, from the
// inner sums (after the barrier that follows them).
template <int ORDER, typename T>
__device__ __forceinline__ void mixed_back(const T* mix_, int w, int lane,
                                           T ihxy, T ihxz, T ihyz, T& dxy,
                                           T& dxz, T& dyz) {
  using F = FD<ORDER>;
  using Geo = SplitGeo<ORDER>;
  using MG = MixGeo<Geo>;
  constexpr int M = MG::M, XW = MG::XW, NX = MG::NX;
  typedef __attribute__((address_space(3))) T lds_t;
  const lds_t* mx = (const lds_t*)mix_;
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int tx = ln & 15, ty = ln >> 4;
  // lowest x tap (x - M) of this point in PX and QX
  const lds_t* px = mx + (w * Geo::TY + ty) * XW + tx;
  asm("" : "+v"(px));
  // y sums at (x, y, z + k): PX inside the tile, PZ on the planes beyond
  const lds_t* pxc = mx + ty * XW + tx + M;
  const lds_t* pzc = mx + 2 * NX + ty * Geo::TX + tx;
  T ta[2 * M], tq[2 * M], td[2 * M];
#pragma unroll
  for (int i = 1; i <= M; ++i) {
    ta[2 * i - 2] = px[M + i];
    ta[2 * i - 1] = px[M - i];
    tq[2 * i - 2] = px[NX + M + i];
    tq[2 * i - 1] = px[NX + M - i];
    const int zp = w + i, zm = w - i;  // uniform
    td[2 * i - 2] = zp < Geo::TZ ? pxc[zp * Geo::TY * XW]
                                 : pzc[(zp - Geo::TZ + M) * Geo::TY * Geo::TX];
    td[2 * i - 1] = zm >= 0 ? pxc[zm * Geo::TY * XW]
                            : pzc[(zm + M) * Geo::TY * Geo::TX];
  }
  T a = T(0), q = T(0), d = T(0);
#pragma unroll
  for (int i = 1; i <= M; ++i) {
    a += T(F::a(i)) * (ta[2 * i - 2] - ta[2 * i - 1]);
    q += T(F::a(i)) * (tq[2 * i - 2] - tq[2 * i - 1]);
    d += T(F::a(i)) * (td[2 * i - 2] - td[2 * i - 1]);
  }
  dxy = a * ihxy;
  dxz = q * ihxz;
  dyz = d * ihyz;
  keep(dxy);
  keep(dxz);
  keep(dyz);
}

// ---- per-tile helpers -------------------------------------------------------------
// Byte offset of the point (x, y, z) in a slot, or beyond every slot for a
// point outside the grid (loads return 0 and stores are dropped there,
// without traffic).
constexpr uint32_t kNoPoint = 0xFFFFFFF0u;
__device__ __forceinline__ uint32_t point_offset(const Patch& P, int x, int y,
                                                 int z) {
  const int g = P.ghost;
  return x < P.n[0] && y < P.n[1] && z < P.n[2]
             ? uint32_t(z + g) * (uint32_t(P.sz) * 8u) +
                   uint32_t(y + g) * (uint32_t(P.sy) * 8u) +
                   uint32_t(x + g) * 8u
             : kNoPoint;
}

// Minimum lapse over the tile's points inside the grid, from cen, in every
// wave alike (as tile_lapse_min).
__device__ __forceinline__ double split_lapse_min(const double* cen,
                                                  const Patch& P, int x0,
                                                  int y0, int z0, int lane) {
  const lds_double* sa = (const lds_double*)cen + 3 * 256;
  const bool in_xy =
      x0 + (lane & 15) < P.n[0] && y0 + (lane >> 4) < P.n[1];
  double a = 1.0e300;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const double v = sa[w * 64 + lane];
    if (in_xy && z0 + w < P.n[2]) a = fmin(a, v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) a = fmin(a, __shfl_xor(a, off, 64));
  return a;
}

// The handed-over sums of a tile whose last step had heavy buffer hp.
template <int ORDER, typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* hand_array(
    SplitLds<ORDER, T>& L, int hp) {
  typedef __attribute__((address_space(3))) T lds_t;
  if constexpr (SplitGeo<ORDER>::HAND_IN_BOX)
    return (lds_t*)((lds_double*)L.heavy + hp * SplitGeo<ORDER>::BUFD);
  else
    return (lds_t*)L.hand;
}

// DMA byte offset of the granule at (xx, yy, zz) of a box (its first element;
// xx even, the box starting at (x0 - R - 1, y0 - R, z0 - R)).  Static grids:
// from the box base, which dma_tile_base gives per tile.  Periodic grids (an
// even number of points in x, so that no granule straddles the wrap): from
// the slot's start, wrapped per axis.  Granules no stencil reads get an offset
// beyond the slot (2^31 and up: out of range with any box base): their LDS
// words fill with zeros, without traffic.
constexpr uint32_t kNoGranule = 0x80000000u;
// c into [0, n); once: -n <= c < 2 n, else c >= -2 n.
__device__ __forceinline__ int wrap(int c, int n, bool once) {
  if (!once) return int(unsigned(c + 2 * n) % unsigned(n));
  c += c < 0 ? n : 0;
  return c - (c >= n ? n : 0);
}
template <class Geo, bool PER>
__device__ __forceinline__ uint32_t granule_offset(const Patch& P, int xx,
                                                   int yy, int zz, bool used,
                                                   int x0, int y0, int z0) {
  if constexpr (PER) {
    // a box ends at most TX + R (TY + R, TZ + R) points beyond the grid: one
    // subtraction wraps it unless the grid is smaller than that (uniform)
    const bool once = P.n[0] >= Geo::TX + Geo::R &&
                      P.n[1] >= Geo::TY + Geo::R && P.n[2] >= Geo::TZ + Geo::R;
    xx = wrap(x0 - Geo::R - 1 + xx, P.n[0], once) + P.ghost;
    yy = wrap(y0 - Geo::R + yy, P.n[1], once) + P.ghost;
    zz = wrap(z0 - Geo::R + zz, P.n[2], once) + P.ghost;
  }
  // (a slot is below 2^31 bytes)
  const uint32_t e = uint32_t(zz) * uint32_t(P.sz) +
                     uint32_t(yy) * uint32_t(P.sy) + uint32_t(xx);
  return used ? e * 8u : kNoGranule;
}
// The granules of a heavy box that this lane moves (instruction j of
// curvature wave w).
template <class Geo, bool PER>
__device__ __forceinline__ void heavy_dma_offsets(const Patch& P, int w,
                                                  int lane, int x0, int y0,
                                                  int z0,
                                                  uint32_t (&off)[Geo::L]) {
#pragma unroll
  for (int j = 0; j < Geo::L; ++j) {
    const int i = (w * Geo::L + j) * 64 + lane;
    const int col = i % (Geo::W / 2), row = i / (Geo::W / 2);
    const int yy = row % Geo::H, zz = row / Geo::H;
    const bool in_y = yy >= Geo::R && yy < Geo::R + Geo::TY;
    const bool in_z = zz >= Geo::R && zz < Geo::R + Geo::TZ;
    const bool in_x = 2 * col + 1 >= Geo::R + 1 && 2 * col <= Geo::R + Geo::TX;
    off[j] = granule_offset<Geo, PER>(P, 2 * col, yy, zz,
                                      i < Geo::G && (in_x || in_y || in_z),
                                      x0, y0, z0);
  }
}
// The same for the runs of a light slot.
template <class Geo, bool PER>
__device__ __forceinline__ void light_dma_offsets(const Patch& P, int w,
                                                  int lane, int x0, int y0,
                                                  int z0,
                                                  uint32_t (&off)[Geo::LL]) {
#pragma unroll
  for (int j = 0; j < Geo::LL; ++j) {
    const int i = ((w * Geo::LL + j) * 64 + lane) * 2;  // element
    int xx, yy, zz;
    if (i < Geo::LX) {
      xx = i % Geo::W;
      const int row = i / Geo::W;
      yy = Geo::R + row % Geo::TY;
      zz = Geo::R + row / Geo::TY;
    } else if (i < Geo::LX + Geo::LY) {
      const int m = i - Geo::LX;
      xx = Geo::R + 1 + m % Geo::TX;
      yy = (m / Geo::TX) % Geo::H;
      zz = Geo::R + m / (Geo::TX * Geo::H);
    } else {
      const int m = i - Geo::LX - Geo::LY;
      xx = Geo::R + 1 + m % Geo::TX;
      yy = Geo::R + (m / Geo::TX) % Geo::TY;
      zz = m / (Geo::TX * Geo::TY);
    }
    off[j] = granule_offset<Geo, PER>(P, xx, yy, zz, i < 2 * Geo::LG, x0, y0,
                                      z0);
  }
}

// ---- the curvature waves ---------------------------------------------------------
template <int ORDER, typename T, bool SKIP, bool PER, class WK>
__device__ __forceinline__ void curvature_waves(const Patch& P, const Gauge& G,
                                                const WK& Wk,
                                                SplitLds<ORDER, T>& S_,
                                                int w, int lane) {
  using Geo = SplitGeo<ORDER>;
  typedef __attribute__((address_space(3))) T lds_t;
  const int n = Wk.count();
  // (scalar, as in Transport)
  const int32_t nbytes = __builtin_amdgcn_readfirstlane(int32_t(P.sf * 8));
  T ih[3], ih2[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ih[a] = T(P.ih[a]);
    ih2[a] = T(P.ih2[a]);
  }
  const T ihxy = T(P.ihm[0]), ihxz = T(P.ihm[1]), ihyz = T(P.ihm[2]);
  const lds_double* heavy0 = (const lds_double*)S_.heavy;
  const lds_double* light0 = (const lds_double*)S_.light;
  // the lane number through an opaque copy: what is derived from it is
  // formed where it is used instead of holding registers through the loop
  auto own_lane = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    return ln;
  };
  auto heavy_taps = [&](const lds_double* hv) {
    const int ln = own_lane();
    return HeavyTaps<ORDER>(hv + (w * Geo::H + (ln >> 4)) * Geo::W +
                            (ln & 15) + 1);
  };
  // DMA of step s of the workgroup's k-th tile (box base tb): its heavy
  // slot, its light slots
  uint32_t hoff[Geo::L], loff[Geo::LL];
  int x0, y0, z0;
  Wk.origin(0, x0, y0, z0);
  heavy_dma_offsets<Geo, PER>(P, w, lane, x0, y0, z0, hoff);
  light_dma_offsets<Geo, PER>(P, w, lane, x0, y0, z0, loff);
  auto issue_heavy = [&](int k, int s, uint32_t tb) {
    const v4i d = slot_dma_rsrc(P.u_s, P.sf, kStepHeavy[s], nbytes);
    const uint32_t l0 = lds_addr(S_.heavy + Geo::heavy_buf(k, s) * Geo::BUFD) +
                        uint32_t(w * Geo::L) * 1024u;
#pragma unroll
    for (int j = 0; j < Geo::L; ++j)
      if (j < Geo::NI - 3 * Geo::L || w < 3)
        dma16(d, PER ? hoff[j] : hoff[j] + tb, l0 + j * 1024u);
  };
  auto issue_light = [&](int k, int s, uint32_t tb) {
#pragma unroll
    for (int i = kStepLight0[s]; i < kStepLight0[s + 1]; ++i) {
      const v4i d = slot_dma_rsrc(P.u_s, P.sf, kStepLight[i], nbytes);
      const uint32_t l0 =
          lds_addr(S_.light + Geo::light_buf(k, i) * Geo::LBUFD) +
          uint32_t(w * Geo::LL) * 1024u;
#pragma unroll
      for (int j = 0; j < Geo::LL; ++j)
        if (j < Geo::LNI - 3 * Geo::LL || w < 3)
          dma16(d, PER ? loff[j] : loff[j] + tb, l0 + j * 1024u);
    }
  };
  // DMA of the transport waves' centre values (wave w: entry w of cen)
  auto issue_centre = [&](uint32_t tb) {
    const v4i d = slot_dma_rsrc(P.u_s, P.sf, kCentreSlots[6] + w,
                                nbytes);
    const v4i da = slot_dma_rsrc(P.u_s, P.sf, ALP, nbytes);
    const uint32_t l0 = lds_addr(S_.cen + w * 256);
    const int ln = own_lane();
    const uint32_t o = uint32_t((int64_t(Geo::R + (ln >> 5)) * P.sz +
                                 int64_t(Geo::R + ((ln >> 3) & 3)) * P.sy +
                                 Geo::R + 1 + 2 * (ln & 7)) * 8) + tb;
    dma16(w < 3 ? d : da, o, l0);
    dma16(w < 3 ? d : da, o + uint32_t(P.sz) * 16u, l0 + 1024u);
  };
  uint32_t tb = dma_tile_base<Geo>(P, x0, y0, z0);
  issue_centre(tb);
  issue_heavy(0, 0, tb);
  issue_light(0, 0, tb);
  if (!Geo::LATE) {
    issue_heavy(0, 1, tb);
    issue_light(0, 1, tb);
  }
  // the metric at the point of the next tile, loaded at the end of a tile
  // (the barrier that follows waits for the next boxes anyway)
  double gn[6];
  auto load_metric = [&](int x, int y, int z) {
    const int ln = own_lane();
    const uint32_t vc =
        point_offset(P, x + (ln & 15), y + (ln >> 4), z + w);
#pragma unroll
    for (int m = 0; m < 6; ++m)
      gn[m] = bload(slot_rsrc(P.u_s, P.sf, GXX + m, nbytes), vc, 0);
  };
  load_metric(x0, y0, z0);
  for (int k = 0; k < n; ++k) {
    int xn = x0, yn = y0, zn = z0;
    if (k + 1 < n) Wk.origin(k + 1, xn, yn, zn);
    const uint32_t tbn = dma_tile_base<Geo>(P, xn, yn, zn);
    const bool more = k + 1 < n;
    // the barrier that opens step s > 0: everything but the DMA issued for
    // later steps has landed (step 10 of the last tile: nothing later)
    auto enter = [&](int s) {
      constexpr int NH0 = Geo::L, NH3 = Geo::NI - 3 * Geo::L;
      constexpr int NL0 = Geo::LL, NL3 = Geo::LNI - 3 * Geo::LL;
      if (s == kNStep - 1 && !more)
        step_barrier<0>();
      else if (Geo::LATE)
        w < 3 ? step_barrier<NH0>() : step_barrier<NH3>();
      else if (n_light((s + 1) % kNStep) == 1)
        w < 3 ? step_barrier<NH0 + NL0>() : step_barrier<NH3 + NL3>();
      else
        w < 3 ? step_barrier<NH0 + 2 * NL0>() : step_barrier<NH3 + 2 * NL3>();
    };
    // DMA issued in step s: after its inner sums, and (LATE) once its box
    // has been read
    // (periodic grids: the lanes' offsets are the next tile's from here on)
    auto fetch = [&](int s) {
      if (PER && more && s == (Geo::LATE ? 10 : 9)) {
        light_dma_offsets<Geo, PER>(P, w, own_lane(), xn, yn, zn, loff);
        if (!Geo::LATE)
          heavy_dma_offsets<Geo, PER>(P, w, own_lane(), xn, yn, zn, hoff);
      }
      if (Geo::LATE) {
        if (s + 1 < kNStep)
          issue_light(k, s + 1, tb);
        else if (more)
          issue_light(k + 1, 0, tbn);
        // (the box of step 1 held the last tile's sums until now)
        if (s == 0) issue_heavy(k, 1, tb);
      } else if (s + 2 < kNStep) {
        issue_heavy(k, s + 2, tb);
        issue_light(k, s + 2, tb);
      } else if (more) {
        issue_heavy(k + 1, s + 2 - kNStep, tbn);
        issue_light(k + 1, s + 2 - kNStep, tbn);
      }
      if (s == 9 && more) issue_centre(tbn);
    };
    auto fetch_late = [&](int s) {
      if (!Geo::LATE) return;
      mid_barrier();
      if (s + 2 < kNStep)
        issue_heavy(k, s + 2, tb);
      else if (s + 2 == kNStep && more) {
        if (PER)
          heavy_dma_offsets<Geo, PER>(P, w, own_lane(), xn, yn, zn, hoff);
        issue_heavy(k + 1, 0, tbn);
      }
    };
    step_barrier<0>();  // step 0
#pragma unroll
    for (int m = 0; m < 6; ++m) keep(gn[m]);
    if constexpr (SKIP) {
      if (split_lapse_min(S_.cen, P, x0, y0, z0, lane) < G.alpha_thr) {
        // left to the FP64 pass: keep the barriers and the DMA going
#pragma unroll
        for (int s = 0; s < kNStep; ++s) {
          if (s > 0) enter(s);
          mid_barrier();
          fetch(s);
          fetch_late(s);
        }
        if (more) load_metric(xn, yn, zn);
        x0 = xn, y0 = yn, z0 = zn;
        tb = tbn;
        continue;
      }
    }
    const lds_double* hv = heavy0;
    T ch;  // the heavy slot's value at the point
    // the two halves of a step: derivatives of the heavy slot
    auto open = [&](int s, T(&d1)[3], T(&d2)[3]) {
      if (s > 0) enter(s);
      hv = heavy0 + Geo::heavy_buf(k, s) * Geo::BUFD;
      inner_sums<ORDER, T, false>(hv, S_.mix, w, lane);
      mid_barrier();
      fetch(s);
      const HeavyTaps<ORDER> t = heavy_taps(hv);
      derivs<ORDER, T, true>(t, ih, ih2, d1, d2);
      ch = T(t.c());
      fetch_late(s);
    };
    auto close = [&](T& dxy, T& dxz, T& dyz) {
      mixed_back<ORDER, T>(S_.mix, w, lane, ihxy, ihxz, ihyz, dxy, dxz, dyz);
    };
    auto light = [&](int i) {
      const LightOffsets<ORDER> lo(w, own_lane());
      return LightTaps<ORDER>(light0 + Geo::light_buf(k, i) * Geo::LBUFD,
                              lo.x, lo.y, lo.z);
    };
    T gt[6], gu[6], dgt[6][3], Rt[6], At[6], none[3];
    auto gamma = [&](int c, int i) {  // d_j Gt^c (light entry i) into R~_ij
      T dG[3];
      derivs<ORDER, T, false>(light(i), ih, ih2, dG, none);
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = p; q < 3; ++q)
          Rt[S(p, q)] += T(0.5) * (gt[S(c, p)] * dG[q] + gt[S(c, q)] * dG[p]);
    };
    constexpr int li[6] = {0, 1, 2, 4, 5, 6};  // A~_ij's light entries
#pragma unroll
    for (int m = 0; m < 6; ++m) gt[m] = T(gn[m]);
    inverse_metric<T>(gt, gu);
#pragma unroll
    for (int m = 0; m < 6; ++m) Rt[m] = T(0);
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      T d2[3], dxy, dxz, dyz;
      open(m, dgt[m], d2);
      At[m] = T(light(li[m]).c());
      if (m == 2) gamma(0, 3);
      if (m == 5) gamma(1, 7);
      close(dxy, dxz, dyz);
      Rt[m] += ricci_trace<T>(gu, d2, dxy, dxz, dyz);
      keep(Rt[m]);
    }
    __builtin_amdgcn_sched_barrier(0);
    T Gu[3][6], Gd[3];
    connection<T, true>(dgt, gu, Gu, Gd, Rt);
    __builtin_amdgcn_sched_barrier(0);
    // phi, with Gt^z
    T dphi[3];
    {
      T dd[6], d2[3];
      open(6, dphi, d2);
      gamma(2, 8);
      close(dd[1], dd[2], dd[4]);
      dd[0] = d2[0];
      dd[3] = d2[1];
      dd[5] = d2[2];
      phi_ricci<T>(gt, gu, Gu, dphi, dd, Rt);
    }
    // alpha, with K
    T Tg[3], rA[6], rK = T(0), trK, alpha;
#pragma unroll
    for (int m = 0; m < 6; ++m) rA[m] = T(0);
    {
      T dal[3], dd[6], d2[3];
      open(7, dal, d2);
      alpha = ch;
      {
        const LightTaps<ORDER> t = light(9);
        T dK[3];
        trK = T(t.c());
        derivs<ORDER, T, false>(t, ih, ih2, dK, none);
#pragma unroll
        for (int i = 0; i < 3; ++i)
          Tg[i] = T(-4.0 / 3.0) * alpha *
                  (gu[S(i, 0)] * dK[0] + gu[S(i, 1)] * dK[1] +
                   gu[S(i, 2)] * dK[2]);
      }
      close(dd[1], dd[2], dd[4]);
      dd[0] = d2[0];
      dd[3] = d2[1];
      dd[5] = d2[2];
      // e^{-4 phi}, left by the transport waves in the last step
      const T em4phi = ((const lds_t*)S_.cen)[w * 64 + own_lane()];
      __builtin_amdgcn_sched_barrier(0);
      lapse_terms<T, true>(gt, gu, Gu, At, Rt, em4phi, dphi, trK, alpha, dal, dd,
                           rA, rK, Tg);
      __builtin_amdgcn_sched_barrier(0);
    }
    // beta^c
    T rg[6], V[3] = {T(0), T(0), T(0)}, divb = T(0);
#pragma unroll
    for (int m = 0; m < 6; ++m) rg[m] = T(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      T db[3], dd[6], d2[3];
      open(8 + c, db, d2);
      close(dd[1], dd[2], dd[4]);
      dd[0] = d2[0];
      dd[3] = d2[1];
      dd[5] = d2[2];
      shift_terms<T>(c, gt, gu, At, Gd, db, dd, rg, rA, Tg, V, divb);
    }
    if (more) load_metric(xn, yn, zn);
    // hand the sums over (the last step's box has been read)
    lds_t* hand = hand_array<ORDER, T>(S_, k & 1) + w * 64 + own_lane();
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      hand[m * 256] =
          rg[m] - T(2) * alpha * At[m] - T(2.0 / 3.0) * gt[m] * divb;
      hand[(6 + m) * 256] = rA[m] - T(2.0 / 3.0) * At[m] * divb;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      hand[(12 + i) * 256] =
          Tg[i] +
          T(1.0 / 3.0) * (gu[S(i, 0)] * V[0] + gu[S(i, 1)] * V[1] +
                          gu[S(i, 2)] * V[2]) -
          T(2.0 / 3.0) * Gd[i] * divb;
    hand[15 * 256] = rK;
    hand[16 * 256] = (divb - alpha * trK) * T(1.0 / 6.0);
    x0 = xn, y0 = yn, z0 = zn;
    tb = tbn;
  }
  step_barrier<0>();  // the last tile's sums
}

// ---- the transport waves ---------------------------------------------------------
template <int ORDER, typename T, bool SKIP, bool KSH>
struct Transport {
  using Geo = SplitGeo<ORDER>;
  typedef __attribute__((address_space(3))) T lds_t;
  const Patch& P;
  const Gauge& G;
  SplitLds<ORDER, T>& S_;
  double* kout;
  const int w, lane;
  const int32_t nbytes;
  int corner;
  LightOffsets<ORDER> lo;
  // the RK4 update as acc = (A or U) + c1 k, out = U + c2 k: what U and A
  // are loaded from and what is stored, by byte range (0: nothing)
  const double* pu;
  int32_t nu, na, nacc;
  bool a_is_u;
  double c1, c2;
  T lapse_f, shift_G, eta;  // 0 where the lapse or the shift is static
  // state
  T cw[3][2 * FD<ORDER>::R];
  T r[NSLOT];
  double U[3], A[3];
  uint32_t vcp = kNoPoint;  // the previous tile's point
  uint32_t vsp = kNoPoint;  // the same on the outermost layer (KSH)
  T q = T(1);

  __device__ __forceinline__ Transport(const Patch& P_, const Gauge& G_,
                                       SplitLds<ORDER, T>& L, int stage,
                                       double* ko, int w_, int lane_)
      : P(P_), G(G_), S_(L), kout(ko), w(w_), lane(lane_),
        nbytes(int32_t(P_.sf * 8)), lo(w_, lane_) {
    const int tx = lane & 15, ty = lane >> 4;
    corner = (w * Geo::H + ty) * Geo::W + tx + 1;
    const double dt = P.dt;
    pu = stage == ST_3 ? P.acc : P.u_n;
    // (uniform, but only readfirstlane makes the compiler hold them in scalar
    // registers: from vector ones every access became a loop over the lanes'
    // descriptors, one after the other: 452 against 376 us for an RK4 step of
    // 83 x 61 x 45, whose workgroups flush after five tiles)
    auto uni = [](int32_t v) { return __builtin_amdgcn_readfirstlane(v); };
    nu = uni(stage == ST_RHS ? 0 : nbytes);
    na = uni(stage == ST_1 || stage == ST_2 ? nbytes : 0);
    nacc = uni(stage == ST_3 || stage == ST_RHS ? 0 : nbytes);
    a_is_u = stage == ST_0;
    c1 = stage == ST_0 ? dt / 6.0 : dt / 3.0;
    c2 = stage == ST_RHS ? 1.0
         : stage == ST_3 ? dt / 6.0
         : stage == ST_2 ? dt
                         : dt / 2.0;
    lapse_f = G.lapse_static ? T(0) : T(G.lapse_f);
    shift_G = G.shift_static ? T(0) : T(G.shift_G);
    eta = G.shift_static ? T(0) : T(G.eta);
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) r[s] = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) U[i] = A[i] = 0.0;
  }

  // loads of the update of step ST's slots at offset vc
  template <int ST, int I = 0>
  __device__ __forceinline__ void update_load(uint32_t vc, double (&u)[3],
                                              double (&a)[3]) const {
    constexpr int s = step_slot(ST, I);
    // (issued also where the stage needs none, with a range of 0 bytes: a
    // branch around them would wait for the loaded value at its end)
    const uint64_t o = slot_bytes(P.sf, s);
    u[I] = bload_nt(rsrc_at(pu, o, nu), vc);
    a[I] = bload_nt(rsrc_at(P.acc, o, na), vc);
    if constexpr (I < n_light(ST)) update_load<ST, I + 1>(vc, u, a);
  }
  template <int ST, int I = 0>
  __device__ __forceinline__ void update_store(const double (&u)[3],
                                               const double (&a)[3]) const {
    constexpr int s = step_slot(ST, I);
    const double k = double(r[s]);
    const uint64_t o = slot_bytes(P.sf, s);
    bstore_nt(rsrc_at(P.acc, o, nacc), vcp,
              (a_is_u ? u[I] : a[I]) + c1 * k);
    bstore_nt(rsrc_at(P.out, o, nbytes), vcp, u[I] + c2 * k);
    if constexpr (KSH) bstore_nt(rsrc_at(kout, o, nbytes), vsp, k);
    if constexpr (I < n_light(ST)) update_store<ST, I + 1>(u, a);
  }

  // the curvature waves' sums of the tile whose last step had heavy buffer hp
  __device__ __forceinline__ void fold(int hp) {
    const lds_t* hand = hand_array<ORDER, T>(S_, hp) + w * 64 + lane;
    constexpr int HS = 256;
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      r[GXX + m] += hand[m * HS];
      r[AXX + m] += hand[(6 + m) * HS];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T t = hand[(12 + i) * HS];
      r[GAMX + i] += t;
      r[BX + i] += G.shift_static ? T(0) : t;
    }
    r[TRK] += hand[15 * HS];
    r[PHI] += hand[16 * HS];
  }

  // step ST of tile k at (x0, y0, z0); vc: the offset of its point
  template <int ST>
  __device__ __forceinline__ void step(int k, int x0, int y0, int z0,
                                       uint32_t vc, bool& skip) {
    mid_barrier();
    if constexpr (SKIP && ST == 0)
      skip = split_lapse_min(S_.cen, P, x0, y0, z0, lane) < G.alpha_thr;
    const lds_double* hv =
        (const lds_double*)S_.heavy + Geo::heavy_buf(k, ST) * Geo::BUFD;
    if (!SKIP || !skip) inner_sums<ORDER, T, true>(hv, S_.mix, w, lane);
    // before the DMA refills the box the sums are in
    if constexpr (ST == 0) fold((k + 1) & 1);
    mid_barrier();
    if constexpr (ST == 0) {
      const lds_double* cen = (const lds_double*)S_.cen + w * 64 + lane;
#pragma unroll
      for (int a = 0; a < 3; ++a)
        axis_weights<ORDER, T>(cen[a * 256], G.ko_eps, P.ih[a], cw[a]);
    }
    T d[3] = {T(0), T(0), T(0)}, c[3] = {T(0), T(0), T(0)};
    if (!SKIP || !skip) {
      const HeavyTaps<ORDER> t(hv + corner);
      d[0] = drift<ORDER, T>(t, cw);
      c[0] = T(t.c());
    }
    // the box has been read: it may be refilled (and holds the tile's sums
    // after the last step)
    if constexpr (Geo::LATE) mid_barrier();
    if (!SKIP || !skip) {
      light_drift<ST, 0>(k, d, c);
      if constexpr (n_light(ST) == 2) light_drift<ST, 1>(k, d, c);
    }
    // e^{-4 phi} for the curvature waves (beta^x's place in cen, which the
    // next tile's takes only at step 9)
    if constexpr (ST == 6) ((lds_t*)S_.cen)[w * 64 + lane] = t_exp<T>(T(-4) * c[0]);
    // the gauge's pointwise terms; K and B^i are set aside where the lapse or
    // the shift is static, as 0 times an infinite one is not 0 (selecting the
    // whole term instead of its factor costs the FMA and 0.5 to 1%)
    if constexpr (ST == 7)
      d[0] -= lapse_f * c[0] * (G.lapse_static ? T(0) : c[1]);
    if constexpr (ST >= 8) {
      if (ST == 8 && G.eta_R > 0.0) {
        const double x = P.origin[0] + (x0 + (lane & 15)) * P.h[0];
        const double y = P.origin[1] + (y0 + (lane >> 4)) * P.h[1];
        const double z = P.origin[2] + (z0 + w) * P.h[2];
        const double rad = sqrt(x * x + y * y + z * z);
        q = T(rad <= G.eta_R ? 1.0 : G.eta_R / rad);
      }
      const T b = G.shift_static ? T(0) : c[1];
      d[0] += shift_G * b;
      d[1] -= eta * q * b;
    }
    // the previous tile's update of this step's slots, and the loads of the
    // next step's: last, when the DMA the curvature waves issued after the
    // barrier has left the address unit free
    update_store<ST>(U, A);
    update_load<(ST + 1) % kNStep>(ST + 1 < kNStep ? vcp : vc, U, A);
    r[kStepHeavy[ST]] = d[0];
    r[kStepLight[kStepLight0[ST]]] = d[1];
    if constexpr (n_light(ST) == 2) r[kStepLight[kStepLight0[ST] + 1]] = d[2];
  }

  // the drift and the centre value of the I-th light slot of step ST
  template <int ST, int I>
  __device__ __forceinline__ void light_drift(int k, T (&d)[3],
                                              T (&c)[3]) const {
    constexpr int e = kStepLight0[ST] + I;
    const LightTaps<ORDER> t(
        (const lds_double*)S_.light + Geo::light_buf(k, e) * Geo::LBUFD, lo.x,
        lo.y, lo.z);
    d[1 + I] = drift<ORDER, T>(t, cw);
    c[1 + I] = T(t.c());
  }

  // the update of every slot of the last tile (step 0's values are loaded)
  template <int ST>
  __device__ __forceinline__ void flush_load(double (&u)[kNStep][3],
                                             double (&a)[kNStep][3]) {
    update_load<ST>(vcp, u[ST], a[ST]);
    if constexpr (ST + 1 < kNStep) flush_load<ST + 1>(u, a);
  }
  template <int ST>
  __device__ __forceinline__ void flush_store(const double (&u)[kNStep][3],
                                              const double (&a)[kNStep][3]) {
    update_store<ST>(u[ST], a[ST]);
    if constexpr (ST + 1 < kNStep) flush_store<ST + 1>(u, a);
  }

  template <class WK>
  __device__ __forceinline__ void run(const WK& Wk) {
    const int n = Wk.count();
    int x0, y0, z0;
    bool skip = false;
    for (int k = 0; k < n; ++k) {
      Wk.origin(k, x0, y0, z0);
      const int x = x0 + (lane & 15), y = y0 + (lane >> 4), z = z0 + w;
      uint32_t vc = point_offset(P, x, y, z);
      step<0>(k, x0, y0, z0, vc, skip);
      if (SKIP && skip) vc = kNoPoint;  // nothing of this tile is written
      step<1>(k, x0, y0, z0, vc, skip);
      step<2>(k, x0, y0, z0, vc, skip);
      step<3>(k, x0, y0, z0, vc, skip);
      step<4>(k, x0, y0, z0, vc, skip);
      step<5>(k, x0, y0, z0, vc, skip);
      step<6>(k, x0, y0, z0, vc, skip);
      step<7>(k, x0, y0, z0, vc, skip);
      step<8>(k, x0, y0, z0, vc, skip);
      step<9>(k, x0, y0, z0, vc, skip);
      step<10>(k, x0, y0, z0, vc, skip);
      vcp = vc;
      if constexpr (KSH) {
        const bool shell = x == 0 || y == 0 || z == 0 || x == P.n[0] - 1 ||
                           y == P.n[1] - 1 || z == P.n[2] - 1;
        vsp = shell ? vc : kNoPoint;
      }
    }
    mid_barrier();
    fold((n - 1) & 1);
    double u[kNStep][3], a[kNStep][3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      u[0][i] = U[i];
      a[0][i] = A[i];
    }
    flush_load<1>(u, a);
    BSSN_PHASE();
    flush_store<0>(u, a);
  }
};

// This thread's wave and lane.  A kernel that calls split_tiles in a loop asks
// for the wave once and never for threadIdx again, which would hold a vector
// register through the calls.
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
}
__device__ __forceinline__ int lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// The tiles Wk names, of patch P.  SKIP: tiles whose minimum lapse is below
// G.alpha_thr are left out (mixed precision's FP32 launch).  KSH: points on
// the outermost interior layer also store their right-hand side to kout.
// PER: periodic grid.  The caller places a barrier before the LDS is used
// again.
template <int ORDER, typename T, bool SKIP, bool KSH, bool PER = false,
          class WK>
__device__ __forceinline__ void split_tiles(const Patch& P, const Gauge& G,
                                            int stage, const WK& Wk,
                                            SplitLds<ORDER, T>& L,
                                            double* kout, int wave) {
  if (Wk.count() <= 0) return;
  // (opaque: a caller's loop over several calls must not keep what both
  // kinds of waves derive from it in registers between them)
  int lane = lane_id();
  asm volatile("" : "+v"(lane));
  if (wave < 4) {
    curvature_waves<ORDER, T, SKIP, PER>(P, G, Wk, L, wave & 3, lane);
  } else {
    Transport<ORDER, T, SKIP, KSH> t(P, G, L, stage, kout, wave & 3, lane);
    t.run(Wk);
  }
}

// ---- kernels ----------------------------------------------------------------------
constexpr int kSplitThreads = 512;

// One patch, FP64: workgroup b takes the tiles of walk_of(b).  KSH: also
// the right-hand side at the outermost interior layer into kout.  PER:
// periodic grid.
template <int ORDER, bool KSH = false, bool PER = false>
__global__ void __launch_bounds__(kSplitThreads)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds(const Patch P, const Gauge G, const int stage,
                const TileMap M, double* const kout) {
  __shared__ __attribute__((aligned(16))) SplitLds<ORDER, double> L;
  split_tiles<ORDER, double, false, KSH, PER>(
      P, G, stage, walk_of(M, gridDim.x), L, kout, wave_id());
}

// Threads of the FP32 launches: at order 4 the FP32 point function fits one
// thread's 256 registers, and two workgroups of 256 threads share a CU
// (lds_tiles); at order 8 it does not, and the split kernel runs it.
template <int ORDER>
constexpr int kF32Threads = ORDER == 8 ? kSplitThreads : 256;

// LDS of an FP32 launch.
template <int ORDER>
struct F32Lds {
  double ring[F32Geo::NBUF * F32Geo::BUFD];
  double sc[kNCentre * 256];
};
template <>
struct F32Lds<8> : SplitLds<8, float> {};

template <int ORDER, bool KSH>
__device__ __forceinline__ void f32_tiles(const Patch& P, const Gauge& G,
                                          int stage, const Walk& w,
                                          F32Lds<ORDER>& L, double* kout) {
  if constexpr (ORDER == 8)
    split_tiles<8, float, true, KSH>(P, G, stage, w, L, kout, wave_id());
  else
    lds_tiles<KSH>(P, G, stage, w, L.ring, L.sc, kout);
}

// One patch, mixed precision, first launch: the FP32 tiles.
template <int ORDER, bool KSH = false>
__global__ void __launch_bounds__(kF32Threads<ORDER>)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds_f32(const Patch P, const Gauge G, const int stage,
                    const TileMap M, double* const kout) {
  __shared__ __attribute__((aligned(16))) F32Lds<ORDER> L;
  f32_tiles<ORDER, KSH>(P, G, stage, walk_of(M, gridDim.x), L, kout);
}

// The tiles of a work item.
__device__ __forceinline__ int item_tiles(const LdsItem& it) {
  return (it.thi - it.tlo + it.stride - 1) / it.stride;
}

// Many patches, mixed precision, first launch: the FP32 tiles, with split
// (1 or 2) workgroups per work list position.  Workgroup b' stands for
// workgroup b of the list's launch of nwg on the same XCD (b' mod 8 = b mod
// 8) and runs part h of every item of b's list.
template <int ORDER>
__global__ void __launch_bounds__(kF32Threads<ORDER>)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds_batch_f32(const Patch* __restrict__ patches,
                          const LdsItem* __restrict__ items,
                          const int32_t* __restrict__ wstart, const Gauge G,
                          const int stage, const int nwg, const int split) {
  __shared__ __attribute__((aligned(16))) F32Lds<ORDER> L;
  const int bp = blockIdx.x;
  const bool xcd = (nwg & 7) == 0;
  const int b = xcd ? 8 * ((bp >> 3) / split) + (bp & 7) : bp / split;
  const int h = xcd ? (bp >> 3) % split : bp % split;
  const int q = walk_pos(b, nwg);
  const int i0 = wstart[q], i1 = wstart[q + 1];
  for (int i = i0; i < i1; ++i) {
    const LdsItem it = items[i];
    const Patch P = patches[it.patch];
    const int n = item_tiles(it);
    const int lo = n * h / split, hi = n * (h + 1) / split;
    const Walk w = walk_dealt(it.tlo + lo * it.stride, hi - lo, it.stride,
                              it.ntx, it.ntz);
    f32_tiles<ORDER, false>(P, G, stage, w, L, nullptr);
    __syncthreads();  // every wave is done with the LDS
  }
}

// Tiles named by an LDS list of tile numbers (TileMap numbering).
typedef __attribute__((address_space(3))) int lds_int;
struct ListWalk {
  const lds_int* t;
  int n, ntx, ntz;
  __device__ __forceinline__ int count() const { return n; }
  __device__ __forceinline__ void origin(int k, int& x0, int& y0,
                                         int& z0) const {
    tile_origin(__builtin_amdgcn_readfirstlane(t[k]), ntx, ntz, x0, y0, z0);
  }
};

// One tile (TileMap numbering), its number held in a register.
struct OneWalk {
  int t, ntx, ntz;
  __device__ __forceinline__ int count() const { return 1; }
  __device__ __forceinline__ void origin(int, int& x0, int& y0,
                                         int& z0) const {
    tile_origin(t, ntx, ntz, x0, y0, z0);
  }
};

// One wave's view of a tile's lapse, four points per lane, read from global
// memory: whether any point is below thr.
struct TileLapse {
  uint32_t o[4];
  double a[4];
  __device__ __forceinline__ void load(const Patch& P, int x0, int y0, int z0,
                                       int lane) {
    const __amdgpu_buffer_rsrc_t r =
        slot_rsrc(P.u_s, P.sf, ALP, int32_t(P.sf * 8));
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      o[z] = point_offset(P, x0 + (lane & 15), y0 + (lane >> 4), z0 + z);
      a[z] = bload(r, o[z], 0);
    }
  }
  __device__ __forceinline__ bool below(double thr) const {
    bool f = false;
#pragma unroll
    for (int z = 0; z < 4; ++z) f = f || (o[z] != kNoPoint && a[z] < thr);
    return __builtin_amdgcn_ballot_w64(f) != 0;
  }
};
constexpr int kScan = 8;  // tiles whose loads a wave has in flight

// Whether the FP64 pass takes tile c of its share (c < hi), below: whether a
// point of it is below thr.  The FP32 launch leaves out the tiles for which the
// minimum of tile_lapse_min and split_lapse_min is below thr.  That minimum
// starts at 1e300 and leaves NaN out: it is below thr where a point is, and
// everywhere if thr exceeds 1e300 (+inf: everything in FP64), also where the lapse
// is NaN at every point.
__device__ __forceinline__ bool fp64_tile(bool below, double thr, int c,
                                          int hi) {
  return below || (thr > 1.0e300 && c < hi);
}

// Writes val of every thread whose flag is set to list, in thread order,
// and returns their number (the same in every thread).  wcnt: 8 ints of
// LDS.  Contains the barriers that make list readable afterwards.
__device__ __forceinline__ int compact_flags(bool f, int val, int wave,
                                             int* list, int* wcnt) {
  const int lane = lane_id();
  const uint64_t mask = __builtin_amdgcn_ballot_w64(f);
  if (lane == 0) wcnt[wave] = __builtin_popcountll(mask);
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSplitThreads / 64; ++w) {
    base += w < wave ? wcnt[w] : 0;
    tot += wcnt[w];
  }
  const int below = __builtin_amdgcn_mbcnt_hi(
      uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
  if (f) list[base + below] = val;
  __syncthreads();
  return tot;
}

// One patch, mixed precision, second launch: the FP64 tiles.  Workgroup b
// examines the tiles t = (i * perm) mod ntiles for i in its share of an
// even split of 0 .. ntiles - 1, a wave taking kScan tiles at a
// time (one tile per thread, a serial walk of its 256 points, made the launch
// 10 us longer: RK4 steps 24^3 263 -> 219 us, 83 x 61 x 45 615 -> 562 us at
// order 4, 97 x 53 x 75 order 8 1,112 -> 1,076 us; 256^3 equal).  perm is
// coprime to ntiles, so every tile is examined exactly once, and the tiles
// around a puncture (neighbours in the numbering) land on many workgroups.
// The tiles whose minimum lapse is below the threshold run through the FP64
// pipeline.
template <int ORDER, bool KSH = false>
__global__ void __launch_bounds__(kSplitThreads)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds_f64tiles(const Patch P, const Gauge G, const int stage,
                         const TileMap M, const int perm,
                         double* const kout) {
  __shared__ __attribute__((aligned(16))) SplitLds<ORDER, double> L;
  __shared__ int list[kSplitThreads];
  // the per-wave counts of compact_flags live in the mixed-derivative
  // scratch, which is idle between split_tiles calls (the LDS is full)
  int* wcnt = (int*)L.mix;
  const int wave = wave_id();
  int lo, hi;
  walk_range(blockIdx.x, gridDim.x, M.ntiles, lo, hi);
  for (int c0 = lo; c0 < hi; c0 += kSplitThreads) {
    // lane l of wave w stands for tile c0 + 8 l + w; the wave examines its
    // lanes' tiles one after the other
    const int lane = lane_id();
    const int c = c0 + 8 * lane + wave;
    const int t = c < hi ? int((int64_t(c) * perm) % M.ntiles) : 0;
    int x0, y0, z0;
    tile_origin(t, M.ntx, M.ntz, x0, y0, z0);
    uint64_t below = 0;
    const int left = hi - c0 - wave;  // tiles c0 + 8 l + wave < hi
    const int nl = left <= 0 ? 0 : (left + 7) / 8 < 64 ? (left + 7) / 8 : 64;
    for (int l0 = 0; l0 < nl; l0 += kScan) {
      TileLapse v[kScan];
#pragma unroll
      for (int i = 0; i < kScan; ++i) {
        const int l = l0 + i < nl ? l0 + i : l0;
        v[i].load(P, __builtin_amdgcn_readlane(x0, l),
                  __builtin_amdgcn_readlane(y0, l),
                  __builtin_amdgcn_readlane(z0, l), lane);
      }
      BSSN_PHASE();
#pragma unroll
      for (int i = 0; i < kScan; ++i)
        below |= uint64_t(l0 + i < nl && v[i].below(G.alpha_thr)) << (l0 + i);
    }
    const bool f = fp64_tile((below >> lane) & 1, G.alpha_thr, c, hi);
    const int n = compact_flags(f, t, wave, list, wcnt);
    if (n > 0) {
      const ListWalk w{(const lds_int*)list, n, M.ntx, M.ntz};
      split_tiles<ORDER, double, false, KSH>(P, G, stage, w, L, kout, wave);
    }
    __syncthreads();  // the LDS, list and wcnt are reused
  }
}

// Many patches, FP64: workgroup b runs the items [wstart[q], wstart[q+1])
// for q = walk_pos(b).
template <int ORDER>
__global__ void __launch_bounds__(kSplitThreads)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds_batch(const Patch* __restrict__ patches,
                      const LdsItem* __restrict__ items,
                      const int32_t* __restrict__ wstart, const Gauge G,
                      const int stage) {
  __shared__ __attribute__((aligned(16))) SplitLds<ORDER, double> L;
  const int wave = wave_id();
  const int q = walk_pos(blockIdx.x, gridDim.x);
  const int i0 = wstart[q], i1 = wstart[q + 1];
  for (int i = i0; i < i1; ++i) {
    const LdsItem it = items[i];
    const Patch P = patches[it.patch];
    const Walk w =
        walk_dealt(it.tlo, item_tiles(it), it.stride, it.ntx, it.ntz);
    split_tiles<ORDER, double, false, false>(P, G, stage, w, L, nullptr, wave);
    __syncthreads();  // every wave is done with the LDS
  }
}

// Many patches, mixed precision, second launch: the FP64 tiles.  Workgroup
// b examines the candidates [lo, hi) of an even split of cand (every tile of
// the launch once, scattered by the plan) as
// k_stage_lds_f64tiles does.
template <int ORDER>
__global__ void __launch_bounds__(kSplitThreads)
    __attribute__((amdgpu_waves_per_eu(2, 2)))
    k_stage_lds_batch_f64tiles(const Patch* __restrict__ patches,
                               const TileRef* __restrict__ cand,
                               const int ncand, const Gauge G,
                               const int stage) {
  __shared__ __attribute__((aligned(16))) SplitLds<ORDER, double> L;
  __shared__ int list[kSplitThreads];
  int* wcnt = (int*)L.mix;  // idle between split_tiles calls
  const int wave = wave_id();
  int lo, hi;
  walk_range(blockIdx.x, gridDim.x, ncand, lo, hi);
  for (int c0 = lo; c0 < hi; c0 += kSplitThreads) {
    const int lane = lane_id();
    const int c = c0 + 8 * lane + wave;
    const TileRef mine = cand[c < hi ? c : lo];
    uint64_t below = 0;
    const int left = hi - c0 - wave;
    const int nl = left <= 0 ? 0 : (left + 7) / 8 < 64 ? (left + 7) / 8 : 64;
    for (int l0 = 0; l0 < nl; l0 += kScan) {
      TileLapse v[kScan];
#pragma unroll
      for (int i = 0; i < kScan; ++i) {
        const int l = l0 + i < nl ? l0 + i : l0;
        const Patch& P = patches[__builtin_amdgcn_readlane(mine.patch, l)];
        const int ntx = (P.n[0] + kLdsTile[0] - 1) / kLdsTile[0];
        const int ntz = (P.n[2] + kLdsTile[2] - 1) / kLdsTile[2];
        int x0, y0, z0;
        tile_origin(__builtin_amdgcn_readlane(mine.tile, l), ntx, ntz, x0, y0,
                    z0);
        v[i].load(P, x0, y0, z0, lane);
      }
      BSSN_PHASE();
#pragma unroll
      for (int i = 0; i < kScan; ++i)
        below |= uint64_t(l0 + i < nl && v[i].below(G.alpha_thr)) << (l0 + i);
    }
    const bool f = fp64_tile((below >> lane) & 1, G.alpha_thr, c, hi);
    const int n = compact_flags(f, c, wave, list, wcnt);
    for (int k = 0; k < n; ++k) {
      const TileRef r = cand[list[k]];
      const Patch P = patches[r.patch];
      const OneWalk w{r.tile, (P.n[0] + kLdsTile[0] - 1) / kLdsTile[0],
                      (P.n[2] + kLdsTile[2] - 1) / kLdsTile[2]};
      split_tiles<ORDER, double, false, false>(P, G, stage, w, L, nullptr, wave);
      __syncthreads();  // every wave is done with the LDS
    }
    __syncthreads();  // the lists and wcnt are reused
  }
}

template <int ORDER>
inline TileMap lds_tile_map(const Patch& P) {
  using Geo = SplitGeo<ORDER>;
  TileMap M;
  M.ntx = (P.n[0] + Geo::TX - 1) / Geo::TX;
  M.nty = (P.n[1] + Geo::TY - 1) / Geo::TY;
  M.ntz = (P.n[2] + Geo::TZ - 1) / Geo::TZ;
  M.ntiles = M.ntx * M.nty * M.ntz;
  M.bx = M.by = M.bz = 0;
  return M;
}

// Blocked walk (Walk with bx > 0) for a launch of 256 or 512 workgroups
// (one or two per CU): the first block shape of nwg / 8 tiles that divides
// the tile grid and gives no workgroup more than 5% more tiles than the even
// split of the dealt walk does (18 block columns on 8 XCDs, a 96^3 grid, would
// cost 29%: 330 against 266 us per order-4 right-hand side; blocks share
// halos in three directions, dealt tiles in z and partly in y and x);
// otherwise the dealt walk.  Order 8
// (a 14-plane box) measured best with blocks 2 tiles deep in z, order 4 with 4.
template <int ORDER>
inline void choose_blocks(TileMap& M, int nwg) {
  static const int s32[][3] = {
      {4, ORDER == 8 ? 4 : 2, ORDER == 8 ? 2 : 4},
      {4, ORDER == 8 ? 2 : 4, ORDER == 8 ? 4 : 2},
      {2, 4, 4}, {2, 2, 8}, {4, 8, 1}, {8, 4, 1}};
  static const int s64[][3] = {{4, 4, 4}, {4, 8, 2}, {8, 4, 2},
                               {2, 8, 4}, {4, 2, 8}, {8, 8, 1}};
  M.bx = M.by = M.bz = 0;
  if (nwg != 256 && nwg != 512) return;
  const int64_t even = (M.ntiles + nwg - 1) / nwg;
  for (const auto& b : (nwg == 256 ? s32 : s64)) {
    if (M.ntx % b[0] || M.nty % b[1] || M.ntz % b[2]) continue;
    const int64_t cols = int64_t(M.ntx / b[0]) * (M.nty / b[1]);
    const int64_t most = (cols + 7) / 8 * (M.ntz / b[2]);
    if (most * 20 > even * 21) continue;
    M.bx = b[0];
    M.by = b[1];
    M.bz = b[2];
    return;
  }
}

// The LDS path needs 16-byte aligned granules: (u + ghost - R - 1) aligned
// and even strides.
template <int ORDER>
inline bool lds_path_ok(const Patch& P) {
  using Geo = SplitGeo<ORDER>;
  const uintptr_t a = reinterpret_cast<uintptr_t>(P.u_s) +
                      8u * uintptr_t(P.ghost - Geo::R - 1);
  return (a % 16) == 0 && (P.sy % 2) == 0 && (P.sz % 2) == 0 &&
         (P.sf % 2) == 0;
}

}  // namespace bssn

namespace bssn {

// The FP64 pass of a mixed-precision stage (k_stage_lds_f64tiles; kout as
// below).  Defined with the batched kernels, whose compiler flags it needs.
template <int ORDER>
hipError_t launch_f64tiles(const Patch& P, const Gauge& G, int stage,
                           const TileMap& M, int nwg, hipStream_t st,
                           double* kout);
template <int ORDER>
inline hipError_t launch_f64tiles_t(const Patch& P, const Gauge& G, int stage,
                                    const TileMap& M, int nwg, hipStream_t st,
                                    double* kout) {
  const int perm = int(tile_perm(M.ntiles));
  if (kout)
    hipLaunchKernelGGL((k_stage_lds_f64tiles<ORDER, true>), dim3(nwg),
                       dim3(kSplitThreads), 0, st, P, G, stage, M, perm, kout);
  else
    hipLaunchKernelGGL((k_stage_lds_f64tiles<ORDER, false>), dim3(nwg),
                       dim3(kSplitThreads), 0, st, P, G, stage, M, perm, kout);
  return hipGetLastError();
}
template <>
hipError_t launch_f64tiles<4>(const Patch&, const Gauge&, int, const TileMap&,
                              int, hipStream_t, double*);
template <>
hipError_t launch_f64tiles<8>(const Patch&, const Gauge&, int, const TileMap&,
                              int, hipStream_t, double*);

// precision 0: one FP64 launch.  Mixed: the FP32 tiles (two workgroups per
// CU at order 4), then the FP64 tiles; both launches take the same per-tile
// decision from the stage input, so each tile is written exactly once.
template <int ORDER, bool KSH>
hipError_t launch_stage_lds_k(const Patch& P, const Gauge& G, int stage,
                              int precision, int nwg_max, hipStream_t st,
                              double* kout) {
  TileMap M = lds_tile_map<ORDER>(P);
  const int nwg = M.ntiles < nwg_max ? M.ntiles : nwg_max;
  if (precision == 0) {
    choose_blocks<ORDER>(M, nwg);
    hipLaunchKernelGGL((k_stage_lds<ORDER, KSH>), dim3(nwg),
                       dim3(kSplitThreads), 0, st, P, G, stage, M, kout);
    return hipGetLastError();
  }
  const int per_cu = ORDER == 4 ? 2 : 1;
  const int nwg32 = M.ntiles < per_cu * nwg_max ? M.ntiles : per_cu * nwg_max;
  TileMap M32 = M;
  choose_blocks<ORDER>(M32, nwg32);
  hipLaunchKernelGGL((k_stage_lds_f32<ORDER, KSH>), dim3(nwg32),
                     dim3(kF32Threads<ORDER>), 0, st, P, G, stage, M32, kout);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_f64tiles<ORDER>(P, G, stage, M, nwg, st, kout);
}
// Periodic grid, FP64.
template <int ORDER>
hipError_t launch_stage_lds_periodic(const Patch& P, const Gauge& G, int stage,
                                     int nwg_max, hipStream_t st) {
  TileMap M = lds_tile_map<ORDER>(P);
  const int nwg = M.ntiles < nwg_max ? M.ntiles : nwg_max;
  choose_blocks<ORDER>(M, nwg);
  hipLaunchKernelGGL((k_stage_lds<ORDER, false, true>), dim3(nwg),
                     dim3(kSplitThreads), 0, st, P, G, stage, M, nullptr);
  return hipGetLastError();
}
// The LDS kernel takes a periodic grid in FP64 with an even number of points
// in x: the boxes' 16-byte granules then wrap as wholes (each lane forms its
// wrapped DMA offsets once per tile).  Odd ones, and mixed precision (whose
// tiles are the direct kernels'), stay on the direct kernels.  Measured, direct
// and here: a 32^3 RK4 step 232 and 102 us, a 96^3 right-hand side 1,330 and
// 330 us (order 4; 266 with the walks as they are now), order 8 3,850 and
// 513 us.
inline bool lds_periodic_ok(const Patch& P, int precision) {
  return precision == 0 && P.n[0] % 2 == 0;
}

// kout set: the kernels that also store the right-hand side at the
// outermost interior layer there.
template <int ORDER>
hipError_t launch_stage_lds(const Patch& P, const Gauge& G, int stage,
                            int precision, int nwg_max, hipStream_t st,
                            double* kout = nullptr) {
  return kout ? launch_stage_lds_k<ORDER, true>(P, G, stage, precision,
                                                nwg_max, st, kout)
              : launch_stage_lds_k<ORDER, false>(P, G, stage, precision,
                                                 nwg_max, st, nullptr);
}

// Explicit-variant launch of one static patch, and batched launches.
template <int ORDER>
hipError_t launch_patch_t(const Patch& P, const Gauge& G, int stage,
                          int precision, int variant, int nwg,
                          hipStream_t st) {
  switch (variant) {
    case VAR_LDS:
      return launch_stage_lds<ORDER>(P, G, stage, precision, nwg, st);
    case VAR_D64:
    case VAR_D64Z4:  // per patch, one plane per workgroup (same results)
      return launch_stage_variant<ORDER, false>(P, G, stage, precision, 64,
                                                st);
    case VAR_D32:
    case VAR_D32Z4:
      return launch_stage_variant<ORDER, false>(P, G, stage, precision, 32,
                                                st);
  }
  return hipErrorInvalidValue;
}

template <int ORDER>
bool variant_ok_t(const Patch& P, int variant) {
  if (variant != VAR_LDS) return variant > VAR_LDS && variant < NVAR;
  Patch q = P;
  const double* bufs[4] = {P.u_s, P.u_n, P.acc, P.out};
  for (const double* b : bufs) {
    if (!b) continue;
    q.u_s = b;
    if (!lds_path_ok<ORDER>(q)) return false;
  }
  return true;
}

template <int ORDER>
hipError_t launch_batch_t(const BatchLaunch& B, const Gauge& G, int stage,
                          int precision, hipStream_t st) {
  if (B.variant == VAR_LDS) {
    const LdsItem* it = static_cast<const LdsItem*>(B.items);
    if (precision == 0) {
      hipLaunchKernelGGL((k_stage_lds_batch<ORDER>), dim3(B.nwg),
                         dim3(kSplitThreads), 0, st, B.patches, it, B.wstart, G, stage);
      return hipGetLastError();
    }
    if (!B.cand) return hipErrorInvalidValue;  // the plan always builds it
    const int split = ORDER == 4 ? 2 : 1;
    hipLaunchKernelGGL((k_stage_lds_batch_f32<ORDER>), dim3(split * B.nwg),
                       dim3(kF32Threads<ORDER>), 0, st, B.patches, it, B.wstart, G, stage,
                       B.nwg, split);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || B.ncand <= 0) return e;
    const int nwg64 = B.ncand < B.nwg ? B.ncand : B.nwg;
    hipLaunchKernelGGL((k_stage_lds_batch_f64tiles<ORDER>), dim3(nwg64),
                       dim3(kSplitThreads), 0, st, B.patches, B.cand, B.ncand, G,
                       stage);
    return hipGetLastError();
  }
  if (B.variant <= VAR_LDS || B.variant >= NVAR) return hipErrorInvalidValue;
  return launch_direct_batch<ORDER>(
      B.patches, static_cast<const DirectItem*>(B.items), B.nitems,
      kVarTile[B.variant][0], kVarTile[B.variant][2], G, stage, precision,
      st);
}

}  // namespace bssn
