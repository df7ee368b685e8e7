// bssn_lds.h -- what the kernels that stage stencil boxes in LDS share (tile
// walks, buffer->LDS DMA, the mixed-derivative layout), and the order-4 FP32
// pipeline of mixed precision.
//
// The pipeline: a workgroup of 256 threads owns one 16 x 4 x 4 tile at a time
// (one thread per point, wave w = z-plane w of the tile).  The point function
// visits the 25 slots one phase at a time (kPhaseSlot order); for each phase
// the haloed box of that slot, (16 + 2R + 1) x (4 + 2R) x (4 + 2R) doubles
// with rows starting one column early so that every 16-byte granule is
// aligned, sits in one of three LDS buffers.  Boxes are fetched with
// buffer_load_dwordx4 ... lds (each lane moves one granule straight into
// LDS, no registers), two phases ahead of use, and the pipeline runs on
// across tile boundaries, so the HBM/L2 latency of one phase hides behind the
// arithmetic of the previous ones.  Stencil taps are then ds_read_b64 /
// ds_read2_b64 with immediate offsets from one per-thread address.  Granules
// a slot's stencils never read are not fetched (their lanes get an offset
// beyond the slot).
//
// Synchronisation per phase: wait until this wave's DMA for the phase has
// landed (an explicit vmcnt: the number of memory instructions the wave
// issued after it), barrier (all waves' granules have landed, and every
// wave is done with the previous phase's buffer), then issue the DMA for
// phase p + NBUF - 1 into the buffer phase p - 1 used.
//
// The FP32 point function fits 256 registers and the ring 80 KB, so that two
// workgroups share a CU and fill each other's waits.  The FP64 one does not:
// it and everything at order 8 run in the split kernels (bssn_split.h).
//
// Mixed precision runs as two launches per stage: k_stage_lds_f32 skips the
// tiles whose minimum lapse is below the threshold; k_stage_lds_f64tiles then
// finds those tiles by the same test and runs them in FP64.
//
// Tiles are walked persistently (Walk): in blocks of 32 (or 64) tiles per
// XCD stepping together in z where the tile grid allows, else dealt in turn to
// an XCD's workgroups, so tiles whose halos overlap are in flight on one XCD and
// meet in its L2.
#pragma once
#include <hip/hip_runtime.h>

#include "bssn_stage.h"

namespace bssn {

// Box and ring geometry of the order-4 FP32 pipeline.  A box of G 16-byte
// granules is moved by 4 L DMA instructions of 64 lanes, L per wave.  A ring
// of three boxes and the centre block take 80 KB.
struct F32Geo {
  static constexpr int R = 3, TX = 16, TY = 4, TZ = 4;
  static constexpr int W = 24;  // (TX + 2R + 1) rounded up to even
  static constexpr int H = TY + 2 * R, D = TZ + 2 * R;
  static constexpr int G = W * H * D / 2;    // granules per box
  static constexpr int L = (G + 255) / 256;  // DMA instructions per wave
  static constexpr int NBUF = 3;             // ring of boxes in LDS
  static constexpr int BUFD = L * 256 * 2;   // doubles per buffer
};
static_assert(F32Geo::TX == kLdsTile[0] && F32Geo::TY == kLdsTile[1] &&
                  F32Geo::TZ == kLdsTile[2],
              "host work lists assume the kLdsTile shape");

// Layout of the shared mixed-derivative scratch (elements of the point
// function's type): PX, the y-sums at the tile's positions extended by MX
// in x ([TZ][TY][TX + 2 MX]); QX, the z-sums at the same positions; PZ, the
// y-sums at the tile's x, y positions on the MX planes below and above the
// tile ([2 MX][TY][TX]).  Every part is a whole number of 64-entry chunks.
template <class Geo>
struct MixGeo {
  static constexpr int M = Geo::MX, XW = Geo::TX + 2 * M;
  static constexpr int NX = Geo::TZ * Geo::TY * XW;  // entries of PX (QX)
  static constexpr int NZ = 2 * M * Geo::TY * Geo::TX;
  static constexpr int NE = 2 * NX + NZ;
  static constexpr int NC = NE / 64;          // chunks
  static_assert(NX % 64 == 0 && NZ % 64 == 0, "whole chunks per part");
};

typedef __attribute__((address_space(3))) double lds_double;

// Per-lane part of the DMA byte offsets (within one slot) of the granules
// this lane moves: the granule's place in the box, independent of the tile.
// The tile adds a wave-uniform byte offset (dma_tile_base), so one set of
// per-lane registers serves every tile.
template <class Geo>
__device__ __forceinline__ void dma_lane_offsets(const Patch& P, int wave,
                                                 int lane,
                                                 uint32_t (&off)[Geo::L]) {
#pragma unroll
  for (int j = 0; j < Geo::L; ++j) {
    const int q = (wave * Geo::L + j) * 64 + lane;
    const int col = q % (Geo::W / 2);
    const int row = q / (Geo::W / 2);
    const int yy = row % Geo::H, zz = row / Geo::H;
    const int64_t e = int64_t(zz) * P.sz + int64_t(yy) * P.sy + 2 * col;
    // Padding lanes (granules past the box) take an offset at or beyond
    // 2^31, so that with any tile base below 2^31 the sum stays out of the
    // slot (slots are < 2^31 bytes): their granules fill the buffer's pad
    // with zeros, without traffic.
    off[j] = q < Geo::G ? uint32_t(e * 8) : 0x80000000u;
  }
}

// Byte offset of the box origin (x0 - R - 1, y0 - R, z0 - R) of the tile
// at interior coordinates (x0, y0, z0), uniform over the workgroup.  The
// one box that starts 8 bytes before the slot (ghost = R, grid corner) has
// base 2^32 - 8: its first granule's first element (the alignment column,
// never read) is out of range, and its second element wraps to offset 0,
// the slot's first element, which it is.
template <class Geo>
__device__ __forceinline__ uint32_t dma_tile_base(const Patch& P, int x0,
                                                  int y0, int z0) {
  const int g = P.ghost;
  const int64_t e = int64_t(z0 + g - Geo::R) * P.sz +
                    int64_t(y0 + g - Geo::R) * P.sy + (x0 + g - Geo::R - 1);
  return __builtin_amdgcn_readfirstlane(uint32_t(e * 8));
}

// One buffer->LDS DMA instruction: every lane moves the 16 bytes at
// `voff` of the buffer described by (base, nbytes) to LDS address
// lds + 16 * lane.  Issued through inline asm so that the compiler's
// conservative LDS-DMA tracking (which cannot tell our ring buffers apart
// once the read pointer is opaque) does not insert vmcnt(0) before every LDS
// read; all waits for these transfers are explicit (pipeline_wait).  The
// instruction writes no register; M0 is set inside the block, with the one
// wait state the M0 -> LDS-DMA dependency needs.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i dma_rsrc(const double* base, int32_t nbytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  v4i r;
  r.x = int(uint32_t(a));
  r.y = int(uint32_t(a >> 32) & 0xffffu);  // stride 0
  r.z = nbytes;
  r.w = kRsrcWord3;
  return r;
}
__device__ __forceinline__ void dma16(v4i r, uint32_t voff, uint32_t lds) {
  // the LDS address is uniform; say so, so that it stays in an SGPR even
  // where a uniform branch around the call hides that from the compiler
  lds = __builtin_amdgcn_readfirstlane(lds);
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %0, %1, 0 offen lds"
      :
      : "v"(voff), "s"(r), "s"(lds)
      : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return uint32_t(reinterpret_cast<uintptr_t>(
      (const __attribute__((address_space(3))) char*)(p)));
}
// (opaque base and stride, as for slot_rsrc)
__device__ __forceinline__ v4i slot_dma_rsrc(const double* u, int64_t sf,
                                             int s, int32_t nbytes) {
  const double* b = u;
  int64_t o = sf;
  asm volatile("" : "+s"(b), "+s"(o));
  return dma_rsrc(b + s * o, nbytes);
}

// Slots whose stencils include mixed second derivatives (gt_ij, phi,
// alpha, beta^i); the others only read the three axis lines through each
// point.
__host__ __device__ constexpr bool needs_mixed(int slot) {
  return (slot >= GXX && slot <= GZZ) || slot == PHI || slot == ALP ||
         (slot >= BETX && slot <= BETZ);
}

// Per-lane mask of the box granules this lane's DMA instructions move that
// a slot's stencils never read: bit j (star-only slots) or 16 + j (slots
// with mixed derivatives) for instruction j.  Star stencils read whole
// rows through the tile (y and z both in the tile), and the tile's x range
// of rows with y or z in the tile; mixed derivatives also read every row
// with y or z in the tile, and the tile's x range of the other rows.  The
// mask depends only on the lane, not on the tile.
template <class Geo>
__device__ __forceinline__ uint32_t dma_skip_mask(int wave, int lane) {
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < Geo::L; ++j) {
    const int q = (wave * Geo::L + j) * 64 + lane;
    const int col = q % (Geo::W / 2);
    const int row = q / (Geo::W / 2);
    const int yy = row % Geo::H, zz = row / Geo::H;
    const bool in_y = yy >= Geo::R && yy < Geo::R + Geo::TY;
    const bool in_z = zz >= Geo::R && zz < Geo::R + Geo::TZ;
    // box column 0 is x0 - R - 1; the tile's x range is columns R+1 .. R+TX
    const bool in_x = 2 * col + 1 >= Geo::R + 1 && 2 * col <= Geo::R + Geo::TX;
    const bool star = (in_y && in_z) || ((in_y || in_z) && in_x);
    const bool mix = in_y || in_z || in_x;
    if (!star) m |= 1u << j;
    if (!mix) m |= 1u << (16 + j);
  }
  return m;
}

// The DMA of slot `slot`'s box into buf; granules the slot never reads get
// an offset beyond the slot (no traffic; their LDS words are not read).
template <class Geo>
__device__ __forceinline__ void dma_issue(const Patch& P, int slot,
                                          double* buf, int wave,
                                          const uint32_t (&off)[Geo::L],
                                          uint32_t tbase, uint32_t skip) {
  static_assert(Geo::L <= 16, "skip mask holds 16 instructions per kind");
  const v4i r = slot_dma_rsrc(P.u_s, P.sf, slot, int32_t(P.sf * 8));
  const uint32_t l0 = lds_addr(buf) + uint32_t(wave * Geo::L) * 1024u;
  const int sh = needs_mixed(slot) ? 16 : 0;
#pragma unroll
  for (int j = 0; j < Geo::L; ++j) {
    const uint32_t o =
        (off[j] + tbase) | ((skip << (31 - (sh + j))) & 0x80000000u);
    dma16(r, o, l0 + j * 1024u);
  }
}

// Centre values the algebra needs before the slot's own phase (gt_ij,
// beta^i, alpha at phase 0) come from a per-tile LDS block (10 slots x 256
// points) that is fetched by DMA one tile ahead, at phase kCentrePhase of
// the previous tile, right after phase 0 read it; ordinary global loads
// would make the in-order vmcnt wait for every prefetch issued before them.
// Other centre values are taken from the slot's own box in its phase.
constexpr int kNCentre = 10;
constexpr int kCentreSlots[kNCentre] = {GXX,  GXY,  GXZ,  GYY, GYZ,
                                        GZZ,  BETX, BETY, BETZ, ALP};
__host__ __device__ constexpr int centre_index(int slot) {
  return slot <= GZZ && slot >= GXX     ? slot - GXX
         : slot >= BETX && slot <= BETZ ? 6 + slot - BETX
                                        : 9;
}
constexpr int kCentrePhase = 1;
constexpr int kCentreL = kNCentre * 128 / 256;  // DMA instructions per wave

// Per-lane DMA offsets of the centre block of the tile at (x0, y0, z0):
// instruction j of wave w moves half of slot kCentreSlots[(5w + j) / 2].
__device__ __forceinline__ void centre_dma(const Patch& P, double* sc,
                                           int x0, int y0, int z0, int wave,
                                           int lane) {
  const int g = P.ghost;
#pragma unroll
  for (int j = 0; j < kCentreL; ++j) {
    const int ins = wave * kCentreL + j;
    const int slot = kCentreSlots[ins >> 1];
    const int within = (ins & 1) * 64 + lane;
    const int row = within >> 3, col = within & 7;
    const int tz = row >> 2, ty = row & 3;
    const int64_t e = int64_t(z0 + tz + g) * P.sz + int64_t(y0 + ty + g) * P.sy +
                      (x0 + g) + 2 * col;
    dma16(slot_dma_rsrc(P.u_s, P.sf, slot, int32_t(P.sf * 8)),
          uint32_t(e * 8), lds_addr(sc) + uint32_t(ins) * 1024u);
  }
}

// s_waitcnt vmcnt(min(N + extra, 63)) lgkmcnt(0) for extra a multiple of
// NSLOT (0 .. 4 NSLOT), rounded down to a value that is never above the
// true count.
template <int N>
__device__ __forceinline__ void vm_wait_n() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N < 63 ? N : 63)
               : "memory");
}
template <int N>
__device__ __forceinline__ void vm_wait_extra(int extra) {
  if (extra <= 0)
    vm_wait_n<N>();
  else if (extra < 2 * NSLOT)
    vm_wait_n<N + NSLOT>();
  else
    vm_wait_n<N + 2 * NSLOT>();
}

// Box element of the lowest tap (y - M for y sums, z - M for z sums) of
// entry `lane` of chunk c of the shared mixed-derivative scratch (MixGeo
// layout).  c is uniform over the wave; the three kinds of chunk (PX, QX,
// PZ) take separate code, so that where c is known at compile time only
// one remains.
template <class Geo>
__device__ __forceinline__ int mix_entry(int c, int lane) {
  using MG = MixGeo<Geo>;
  constexpr int M = MG::M, XW = MG::XW, R = Geo::R, W = Geo::W, H = Geo::H;
  if (c < 2 * MG::NX / 64) {  // PX (y sums) or QX (z sums), x-extended
    // entry i = q XW + ix with q = tz TY + ty: its box element is
    // tz (H W) + ty W + ix + const = tz (H - TY) W + q (W - XW) + i + const
    const bool qx = c >= MG::NX / 64;
    const unsigned i =
        unsigned((qx ? c - MG::NX / 64 : c) * 64) + unsigned(lane);
    const unsigned q = i / unsigned(XW), tz = q / unsigned(Geo::TY);
    constexpr int C0 = (R * H + R - M) * W + R + 1 - M;  // PX: (R, R - M)
    constexpr int C1 = ((R - M) * H + R) * W + R + 1 - M;  // QX: (R - M, R)
    return int(tz * unsigned((H - Geo::TY) * W) + q * unsigned(W - XW) + i) +
           (qx ? C1 : C0);
  }
  // PZ: y sums on the planes beyond the tile; a chunk is one plane
  static_assert(Geo::TX * Geo::TY == 64, "one PZ plane per chunk");
  const int pz = c - 2 * MG::NX / 64;
  const int zr = pz < M ? pz - M : Geo::TZ + pz - M;
  return ((zr + R) * H + (lane >> 4) + R - M) * W + (lane & 15) + R + 1;
}

// Distinct empty asm at both ends of each code path of a uniform branch,
// so that the compiler keeps the paths apart (each with its own immediate
// LDS offsets) instead of merging them into one with selected addresses.
template <int K>
__device__ __forceinline__ void path_mark();
template <>
__device__ __forceinline__ void path_mark<0>() {
  asm volatile("; path 0");
}
template <>
__device__ __forceinline__ void path_mark<1>() {
  asm volatile("; path 1");
}

// Loader used by point_rhs inside the pipelined kernel.  Phase p of the
// k-th tile of a workgroup is global phase k*NSLOT + p and uses ring buffer
// (k*NSLOT + p) mod NBUF.
struct LdLds {
  using Geo = F32Geo;
  const Patch* P;
  double* ring;            // NBUF buffers of BUFD doubles
  double* sc;              // centre block
  const uint32_t* off;     // per-lane DMA offsets within a box
  uint32_t tb_cur, tb_nxt;  // box base of this tile and of the next one
  int nxt[3];              // next tile's origin (centre block prefetch)
  int pbase;               // (k * NSLOT) mod NBUF
  int wave, lane, tid;
  uint32_t skip;           // dma_skip_mask of this lane
  int cidx;                // element index in a box of the thread's stencil
                           // corner (x-R, y-R, z-R)
  int prev_mem;            // memory instructions of the previous tile's
                           // epilogue stores in this wave (0 at the first)
  // this thread's cidx in the current phase's buffer; set per phase
  // through an opaque move so the compiler derives every tap from this one
  // register with immediate offsets instead of hoisting (and spilling) a
  // base address per buffer out of the tile loop
  mutable const lds_double* pc;

  __device__ __forceinline__ double* buffer(int p) const {
    return ring + ((pbase + p) % Geo::NBUF) * Geo::BUFD;
  }
  __device__ __forceinline__ double g(int s) const {
    return ((const lds_double*)sc)[centre_index(s) * 256 + tid];
  }
  __device__ __forceinline__ void enter(int s) const {
    const int p = phase_of(s);
    if (p != 0) phase(p);  // the kernel runs phase 0 itself
    const lds_double* b = (const lds_double*)buffer(p) + cidx;
    asm volatile("" : "+v"(b));
    pc = b;
  }
  // one pipeline step at phase p (0 <= p < NSLOT)
  __device__ __forceinline__ void phase(int p) const {
    // Wait until this wave's DMA for phase p has landed.  vmcnt counts
    // this wave's memory instructions in issue order, so the count to wait
    // for is the number issued after that DMA: the prefetches of phases
    // p+1 .. p+NBUF-2; for phases 2 .. NBUF the centre block issued at
    // phase 1; and at phases 0 .. NBUF-2 of every tile but the first, the
    // previous tile's epilogue stores.  The field holds at most 63, and
    // waiting for fewer than that number is always correct.  lgkmcnt(0):
    // this wave's reads of the buffer about to be refilled have completed.
    const int extra = p <= Geo::NBUF - 2 ? prev_mem : 0;
    if (p > kCentrePhase && p <= kCentrePhase + Geo::NBUF - 1)
      vm_wait_extra<(Geo::NBUF - 2) * Geo::L + kCentreL>(extra);
    else
      vm_wait_extra<(Geo::NBUF - 2) * Geo::L>(extra);
    __builtin_amdgcn_s_barrier();
    const int q = p + Geo::NBUF - 1;  // phase to prefetch
    uint32_t o[Geo::L];
#pragma unroll
    for (int j = 0; j < Geo::L; ++j) o[j] = off[j];
    if (q < NSLOT)
      dma_issue<Geo>(*P, kPhaseSlot[q], buffer(q), wave, o, tb_cur, skip);
    else
      dma_issue<Geo>(*P, kPhaseSlot[q - NSLOT], buffer(q), wave, o, tb_nxt,
                     skip);
    if (p == kCentrePhase)
      centre_dma(*P, sc, nxt[0], nxt[1], nxt[2], wave, lane);
  }
  __device__ __forceinline__ int str(int a) const {
    return a == 0 ? 1 : (a == 1 ? Geo::W : Geo::W * Geo::H);
  }
  // pc is the thread's stencil corner, so every tap is a non-negative
  // immediate offset (fewer address adds, more ds_read2 pairs)
  static constexpr int kC = Geo::R * (1 + Geo::W + Geo::W * Geo::H);
  __device__ __forceinline__ double c(int) const { return pc[kC]; }
  __device__ __forceinline__ double ax(int, int a, int k) const {
    return pc[kC + k * str(a)];
  }
  __device__ __forceinline__ double pl(int, int a, int i, int b, int j) const {
    return pc[kC + i * str(a) + j * str(b)];
  }
};

// Tile walk.  Tiles are numbered z fastest within an (x, y) column:
// t = iz + ntz * (ix + ntx * iy).  Each XCD (workgroups are dispatched
// round-robin: b, b+8, ...) owns a contiguous eighth of them and deals it to
// its workgroups in turn, so that at any time it works on as many neighbouring
// tiles as it has workgroups, whose halos meet in its L2.  With a contiguous
// range per workgroup instead, the tiles in work on an XCD lie far apart: RK4
// steps of 200 x 180 x 160 9.1 against 7.7 ms (order 4), 97 x 53 x 75 order 8
// mixed 1,090 against 1,025 us, 48 uneven patches 17.1 against 14.8 ms.
struct TileMap {
  int ntx, nty, ntz, ntiles;
  int bx, by, bz;  // block shape of the blocked walk, bx = 0: dealt
};
__host__ __device__ __forceinline__ int walk_pos(int wg, int nwg) {
  return (nwg & 7) == 0 ? (wg & 7) * (nwg >> 3) + (wg >> 3) : wg;
}
__host__ __device__ __forceinline__ void walk_range(int lin, int nwg,
                                                    int ntiles, int& lo,
                                                    int& hi) {
  lo = int((int64_t(ntiles) * lin) / nwg);
  hi = int((int64_t(ntiles) * (lin + 1)) / nwg);
}

// Origin (interior coordinates) of tile t of the TileMap numbering.
__device__ __forceinline__ void tile_origin(int t, int ntx, int ntz, int& x0,
                                            int& y0, int& z0) {
  const int iz = t % ntz, col = t / ntz;
  x0 = (col % ntx) * kLdsTile[0];
  y0 = (col / ntx) * kLdsTile[1];
  z0 = iz * kLdsTile[2];
}

// The tiles one workgroup visits, in order (one walker type, so the
// right-hand side is inlined once).  Tile k is c = k / nk, kz = k mod nk:
//   dealt walk (bx = 0): tiles tlo + k stride of the TileMap numbering (z
//     fastest within an (x, y) column), where the workgroups of one XCD hold
//     stride neighbouring tiles at a time; nk = count, c = 0;
//   blocked walk (single patches whose tile grid divides into blocks of
//     bx x by x bz = 32 tiles, or 64 with two workgroups per CU): the
//     workgroups of one XCD hold one tile each of a block, step through
//     the block's column together in z by
//     bz tiles, then move on to the XCD's next block (blocks c*8 + xcd).
//     Neighbouring tiles in x, y and z are then fetched at the same time on
//     one XCD, and between two z-steps the L2 only has to keep the overlap
//     planes of a (16 bx + 2R) x (4 by + 2R) footprint.
struct Walk {
  int n;            // tiles this workgroup visits
  int lx, ly, lz;   // this workgroup's tile within a block
  int bx, by, bz;   // block shape in tiles (bx = 0: dealt walk)
  int xcd, nrx, nk;
  // (the dealt walk's first tile, stride, ntx and ntz share the fields of the
  // blocked one: fewer scalar registers through the tile loop)
  __device__ __forceinline__ int count() const { return n; }
  __device__ __forceinline__ void origin(int k, int& x0, int& y0,
                                         int& z0) const {
    if (bx == 0) {
      tile_origin(xcd + k * nk, nrx, lz, x0, y0, z0);
    } else {
      const int r = xcd + 8 * (k / nk), kz = k % nk;
      x0 = ((r % nrx) * bx + lx) * kLdsTile[0];
      y0 = ((r / nrx) * by + ly) * kLdsTile[1];
      z0 = (kz * bz + lz) * kLdsTile[2];
    }
  }
};
__device__ __forceinline__ Walk walk_dealt(int tlo, int n, int stride,
                                           int ntx, int ntz) {
  Walk w{};
  w.n = n;
  w.xcd = tlo;
  w.nk = stride;
  w.nrx = ntx;
  w.lz = ntz;
  w.bx = 0;
  return w;
}

// Minimum lapse over the tile's points, taken from the centre block (which
// holds all 256 of them) in every wave, so that each wave reaches the same
// value without a barrier.  Points outside the grid do not count.  fmin is
// exact, so the value does not depend on the order of reduction; the FP64
// pass takes the same decision from global memory, point by point (TileLapse).
__device__ __forceinline__ double tile_lapse_min(const double* sc,
                                                 const Patch& P, int x, int y,
                                                 int z0, int lane) {
  const lds_double* sa = (const lds_double*)sc + centre_index(ALP) * 256;
  double a = 1.0e300;
  const bool in_xy = x < P.n[0] && y < P.n[1];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const double v = sa[w * 64 + lane];
    if (in_xy && z0 + w < P.n[2]) a = fmin(a, v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) a = fmin(a, __shfl_xor(a, off, 64));
  return a;
}

// The tiles Wk names, of patch P, in FP32, pipelined through the workgroup's
// LDS ring; tiles whose minimum lapse is below G.alpha_thr run through the
// pipeline without arithmetic.  KSH: a point on the outermost interior layer
// (shell) also stores its right-hand side to kout (the radiative boundary's
// roots, state layout); the stores follow the epilogue's.  On return every
// DMA of this call has landed; the caller places a barrier before the ring is
// filled again.
template <bool KSH, class WK>
__device__ __forceinline__ void lds_tiles(const Patch& P, const Gauge& G,
                                          const int stage, const WK& Wk,
                                          double* ring, double* sc,
                                          double* kout) {
  using Geo = F32Geo;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int tx = lane & 15, ty = lane >> 4, tz = wave;
  const int ntile_mine = Wk.count();
  if (ntile_mine <= 0) return;
  uint32_t off[Geo::L];
  dma_lane_offsets<Geo>(P, wave, lane, off);
  int x0, y0, z0, xn, yn, zn;
  Wk.origin(0, x0, y0, z0);
  uint32_t tbA = dma_tile_base<Geo>(P, x0, y0, z0);
  Wk.origin(ntile_mine > 1 ? 1 : 0, xn, yn, zn);
  uint32_t tbB = dma_tile_base<Geo>(P, xn, yn, zn);
  // DMA only the granules each slot reads (the out-of-range lanes still
  // cost their address slot)
  const uint32_t skip = dma_skip_mask<Geo>(wave, lane);
  // prologue: centre block and phases 0 .. NBUF-2 of the first tile
  centre_dma(P, sc, x0, y0, z0, wave, lane);
#pragma unroll
  for (int q = 0; q < Geo::NBUF - 1; ++q)
    dma_issue<Geo>(P, kPhaseSlot[q], ring + q * Geo::BUFD, wave, off, tbA,
                   skip);

  const int32_t nbytes = int32_t(P.sf * 8);
  const uint32_t sy8 = uint32_t(P.sy) * 8u, sz8 = uint32_t(P.sz) * 8u;
  int prev_mem = 0;  // this wave's last epilogue
  for (int k = 0; k < ntile_mine; ++k) {
    Wk.origin(k, x0, y0, z0);
    const int x = x0 + tx, y = y0 + ty, z = z0 + tz;
    const bool active = x < P.n[0] && y < P.n[1] && z < P.n[2];
    const bool shell = KSH && (x == 0 || y == 0 || z == 0 || x == P.n[0] - 1 ||
                               y == P.n[1] - 1 || z == P.n[2] - 1);
    const int g = P.ghost;
    LdLds ld;
    ld.P = &P;
    ld.ring = ring;
    ld.sc = sc;
    ld.off = off;
    ld.tb_cur = tbA;
    ld.tb_nxt = tbB;
    ld.nxt[0] = xn;
    ld.nxt[1] = yn;
    ld.nxt[2] = zn;
    ld.pbase = (k * NSLOT) % Geo::NBUF;
    ld.wave = wave;
    ld.lane = lane;
    ld.tid = tid;
    ld.skip = skip;
    ld.prev_mem = prev_mem;
    ld.cidx = (tz * Geo::H + ty) * Geo::W + tx + 1;
    // inactive lanes load from and store to beyond the buffer: no traffic,
    // value 0
    const uint32_t vc = active ? uint32_t(z + g) * sz8 + uint32_t(y + g) * sy8 +
                                     uint32_t(x + g) * 8u
                               : 0xFFFFFFF0u;
    ld.phase(0);  // phase 0's box and this tile's centre block have landed
    const double xc = P.origin[0] + x * P.h[0];
    const double yc = P.origin[1] + y * P.h[1];
    const double zc = P.origin[2] + z * P.h[2];
    prev_mem = 0;
    if (tile_lapse_min(sc, P, x, y, z0, lane) < G.alpha_thr) {
      // left to the FP64 pass: keep the pipeline going (waits, barriers,
      // prefetches) through the tile's other phases
#pragma unroll
      for (int p = 1; p < NSLOT; ++p) ld.phase(p);
    } else {
      float r[NSLOT];
      point_rhs<4, float>(ld, P, xc, yc, zc, G, r);
      epilogue_all<float>(P, stage, r, vc, nbytes);
      // every lane loads and stores; the waits count them (the loads too:
      // they follow the DMA of the next tile's first phases)
      prev_mem = epilogue_loads(stage) + epilogue_stores(stage);
      if constexpr (KSH) {
        if (active && shell) {
#pragma unroll
          for (int s = 0; s < NSLOT; ++s)
            bstore_nt(slot_rsrc(kout, P.sf, s, nbytes), vc, double(r[s]));
        }
        // (a wave whose lanes all skip them may still issue them with no
        // lane enabled, which only makes the next waits longer than needed)
        if (__builtin_amdgcn_ballot_w64(active && shell) != 0)
          prev_mem += NSLOT;
      }
    }
    // next tile: its box base becomes current, prepare the one after
    tbA = tbB;
    if (k + 2 < ntile_mine) {
      Wk.origin(k + 2, xn, yn, zn);
      tbB = dma_tile_base<Geo>(P, xn, yn, zn);
    }
  }
  // drain outstanding DMA (the last tile prefetched a next one that is not
  // used) and this wave's LDS reads
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// The walk of workgroup blockIdx.x of a launch of nwg workgroups over M.
__device__ __forceinline__ Walk walk_of(const TileMap& M, int nwg) {
  Walk w{};
  if (M.bx > 0) {
    w.xcd = blockIdx.x & 7;
    const int l = blockIdx.x >> 3;
    w.lx = l % M.bx;
    w.ly = (l / M.bx) % M.by;
    w.lz = l / (M.bx * M.by);
    w.bx = M.bx;
    w.by = M.by;
    w.bz = M.bz;
    w.nrx = M.ntx / M.bx;
    w.nk = M.ntz / M.bz;
    const int nblk = w.nrx * (M.nty / M.by);
    w.n = (nblk > w.xcd ? (nblk - w.xcd + 7) / 8 : 0) * w.nk;
  } else {
    // the tiles of the XCD's share, dealt to its workgroups in turn (without
    // whole XCDs: of the launch)
    const int ngrp = (nwg & 7) == 0 ? 8 : 1, W = nwg / ngrp;
    int lo, hi;
    walk_range(blockIdx.x % ngrp, ngrp, M.ntiles, lo, hi);
    lo += blockIdx.x / ngrp;
    w = walk_dealt(lo, lo < hi ? (hi - lo + W - 1) / W : 0, W, M.ntx, M.ntz);
  }
  return w;
}

}  // namespace bssn
