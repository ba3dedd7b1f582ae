// TV pass kernels of the fused-lasso proximal operator on gfx950: gradient projection on the dual of
// 3D isotropic TV denoising (Beck & Teboulle), then the soft threshold.
//
// With D the forward-difference operator along x, y, z (last difference on
// each axis zero) and u = v - tau D^T p, each dual step is
//     q = p + D u / (12 tau),   p = q / max(1, |q|)
// from p = 0; the result is soft(v - tau D^T p, step*l1).  -D^T p is the
// backward-difference divergence: div p(i) = sum_a p_a(i) - p_a(i - e_a), with
// p_a(i - e_a) = 0 on the first index and p_a = 0 on the last index of axis a.
//
// Temporal blocking.  A dual step at voxel i reads the previous dual at
// offsets in {-1, 0, 1} per axis, so L fused steps need an L-voxel halo.  A
// block owns a 64 x (W Q) tile in (x, y) -- one wavefront lane per x, Q = 4
// rows of y per lane, W = 12 wavefronts stacked in y -- and streams through z
// (one block per CU at up to 170 VGPRs).  The L steps
// form a pipeline along z: step l consumes the dual of step l-1 one plane
// behind it (step 2 two planes behind step 1) and keeps in registers, per
// point, the previous plane's dual and primal values.  A plane costs about 600
// vector operations a wave and three waves a unit hide little, so what bounds a
// pass is the latency of each step's exchange; steps 0 and 2, then 1 and 3, run
// between the same two barriers and fill each other's (1024^2 x 256, 20 steps:
// depth 4 11.24 -> 10.40 ms in 3D, 8.68 -> 7.32 ms in 2D; 512^2 x 128, depth 3
// 2250 -> 2208 and 1285 -> 1219 us; against one barrier per step and plane).  Neighbours along x move with DPP wave shifts, along y through
// registers within a lane and through LDS rows between
// wavefronts.  A kernel compiled for up to H
// fused steps has an H-voxel halo: points within H of the tile edge are
// computed but not stored, and tiles overlap by 2H.  The z-range is cut into
// chunks with an L+1 plane margin so that the grid fills the device.
//
// Per-plane 2D TV (TV2): the TV of the paper's Eq. (4) taken in every plane on
// its own.  The dual has no z component (neither read nor stored), the step is
// 1/(8 tau) and planes do not couple, so chunks need no z margin.
//
// Dual storage in bfloat16 (dual_bf16): the dual between passes is rounded to
// bfloat16 (to nearest, ties to even) when stored and widened when read; the
// arithmetic stays FP32.  The dual lies in the unit ball, so its bytes halve
// at 2^-9 relative precision.
//
// FGP (accelerated dual iteration): every dual pass takes one step at the
// extrapolated point r, reads (r, p_prev) and stores (p, r_next), r_next =
// p + w (p - p_prev) with w = (t_k - 1)/t_{k+1} of the FISTA sequence (set per
// pass by the host); the final pass steps at r like a plain pass.
//
// Boundaries: the z-component of the dual is exactly zero on the last plane
// (its z-difference is zero there, from p = 0 on) and the state below the first
// plane starts at zero, so the divergence carries no z masks; x / y masks are
// compiled only into the blocks whose tile touches the volume edge.
//
// One pass fuses up to H steps; a prox is a sequence of passes ping-ponging the
// dual between two buffers.  The last pass adds a half step (primal recovery),
// the soft threshold, the occupancy flags of the result and the store of x.
// It runs its own kernel whose tile has an (H+1)-voxel halo: x at a voxel needs
// the dual one voxel below it on every axis, and the objective's differences
// need x one voxel above, so with one more voxel of halo the last pass fuses
// a full H dual steps as well (K steps take ceil(K/H) passes).
#pragma once
#include <algorithm>
#include <type_traits>
#include <vector>

#include "rihvr_internal.h"

// A product followed by a sum must round the same way wherever it is compiled:
// the steady and the single-plane form of the pipeline, interior and edge tiles
// and every chunking give the same bits.
#pragma clang fp contract(off)

namespace rihvr {

constexpr int kTvWaves = 12;
constexpr int kTvQ = 4;                 // rows per lane
constexpr int kTvRX = 64;               // tile width (lanes)
constexpr int kTvRY = kTvWaves * kTvQ;  // tile height
constexpr int kTvSmallQ = 2;            // rows per lane of the low tiles (see pass_grid)
template <int Q>
using TvVec = float __attribute__((ext_vector_type(Q)));

struct TvPassArgs {
  const float* v;                 // nullptr: vol[st->prev]
  float* x;                       // nullptr: vol[st->next]
  float* vol[3];
  const float* pin[3];            // dual read by the first step (ignored when first)
  float* pout[3];                 // dual written by the last step (unless final)
  uint8_t* rowflag; uint8_t* planeflag;  // final pass: set where x != 0 (nullable)
  double* psum; double* ptv;      // final pass: per-block sum(x) and TV(x) of the stored x, two words each (nullable)
  const SolveState* st;
  int nx, ny, nz;
  int levels;                     // fused dual steps in this pass (<= H)
  int first, final_, nonneg;
  int tv2;                        // per-plane 2D TV (no z component, no z margin)
  int keep_dual;                  // final pass: also store the dual to pout (warm start of the next prox)
  int flip_npass;                 // > 0: the solve's passes ping-pong the dual across outer iterations;
                                  // pin and pout trade places when (st->it - 1) * flip_npass is odd
  int dual_bf16;                  // the dual buffers hold bfloat16
  const float* pin2[3];           // FGP: p_prev read with r (= pin)
  float* pout2[3];                // FGP: p written beside r_next (= pout)
  float fgp_w;                    // FGP: extrapolation weight of this pass
  RowStores rs;                   // final pass with rs.on: x_{k+1} into row store st->scur ^ 1
  int fgp;                        // FGP dual pass (one step; never the final pass)
  int zchunk;                     // output planes per block (the first nfull tiles)
  int nfull;                      // tiles (in raster order) cut into chunks of zchunk planes; the
  int zchunk2;                    // remaining gx*gy - nfull tiles are cut into chunks of zchunk2
  int nblocks;                    // blocks of the pass (the objective partials are per block)
  float tau, c, thr;
  int gx, gy;                     // tiles along x and y (the grid of one frame)
  int low;                        // tiles of kTvSmallQ rows a lane
  int depth;                      // fusion depth of the kernel that runs the pass
  int seq;                        // ... and its form (TvForm)
  size_t zoff_v, zoff_x;          // grouped per-plane prox: first plane of the group in v and x (elements)
};

// A register copy the compiler keeps (an identity DPP move).  The prefetched
// plane is copied out of its registers before they are reloaded; left to
// itself, the compiler renames the consumer onto the loaded registers, loads
// the next plane into fresh ones and moves them back at the loop's back edge,
// which waits for every load in flight.
__device__ __forceinline__ float vcopy(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xE4, 0xf, 0xf, false));
}
__device__ __forceinline__ float dpp_from_left(float v) {   // lane i <- lane i-1 (0 at lane 0)
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_from_right(float v) {  // lane i <- lane i+1 (0 at lane 63)
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
}

// Planes are addressed through buffer resources: a scalar descriptor of one
// plane (base, size in bytes) and a 32-bit per-lane byte offset.  A load at an
// offset past the plane returns 0 and a store there is dropped, so lanes
// outside the volume or outside the stored region use kTvOff (planes end far
// below it, and the sum of two does not wrap).
constexpr unsigned kTvOff = 0x40000000u;
constexpr int kTvRsrcWord3 = 0x00020000;  // 32-bit data format, no stride / swizzle
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const float* base, size_t plane, size_t sz) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base) + plane * sz, (short)0, (int)(sz * 4),
                                           kTvRsrcWord3);
}
__device__ __forceinline__ float buf_ld(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, unsigned off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)off, 0, 0);
}

// Dual planes, FP32 or bfloat16 (`bf`, uniform).  Offsets are those of the
// FP32 layout; a bfloat16 element sits at half of it (kTvOff / 2 is still past
// every plane).  zero: an empty descriptor, every load returns 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dual_rsrc(const float* base, size_t plane, size_t sz, bool bf,
                                                            bool zero = false) {
  const char* b = reinterpret_cast<const char*>(base) + plane * sz * (bf ? 2 : 4);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(b), (short)0, zero ? 0 : (int)(sz * (bf ? 2 : 4)),
                                           kTvRsrcWord3);
}
// The loaded bits; dual_val makes the value of them where it is used.  (Widened here,
// the shift waits for the loads of a plane that is not needed before the next one:
// prox of 10 steps at depth 3, 512^2 x 128, 1822 us; 894 so.)
__device__ __forceinline__ float dual_ld(__amdgpu_buffer_rsrc_t r, unsigned off, bool bf) {
  if (!bf) return buf_ld(r, off);
  return __uint_as_float((unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(off >> 1), 0, 0));
}
__device__ __forceinline__ float dual_val(float bits, bool bf) {
  const float v = vcopy(bits);
  return bf ? __uint_as_float(__float_as_uint(v) << 16) : v;
}
__device__ __forceinline__ void dual_st(__amdgpu_buffer_rsrc_t r, unsigned off, float v, bool bf) {
  if (!bf) {
    buf_st(r, off, v);
    return;
  }
  const unsigned u = __float_as_uint(v);
  const unsigned h = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;   // round to nearest, ties to even (|v| <= 1)
  __builtin_amdgcn_raw_buffer_store_b16((unsigned short)h, r, (int)(off >> 1), 0, 0);
}

// Pass body.  H: the halo (tile geometry); LV: register slots for fused steps
// (the halo on dual passes; on the final pass, whose halo is one wider, H - 1).  EDGE: the tile
// touches the volume boundary, so every access and every difference is masked;
// interior tiles (most of them) skip the masks.  TV2: per-plane 2D TV.  FINAL: the last pass (primal recovery and output)
// instead of storing the dual.  FGP: a one-step accelerated dual pass (above).
//
// With psum / ptv set, the final pass also sums x and its isotropic TV (forward
// differences, zero at the last index of each axis) over the points it stores.
// The differences of a plane need the next plane, so a plane's terms are taken
// when the next one is output (the last plane of the volume after the loop);
// the x+1 neighbour comes by a wave shift, the y+1 neighbour from the next row
// of the lane or, for the last row, from the next wave through LDS.  Every
// neighbour lies in the computed tile: the final pass fuses at most H - 1
// steps for its halo of H, so x is exact one point beyond the stored region.

// Planes between a plane's arrival and its output after L fused steps: one per
// step, and one more from the third step on (see the pipeline below).
__host__ __device__ constexpr int tv_delay(int L) { return L + (L > 2 ? 1 : 0); }
// Depth 4 keeps what it can out of registers: its final pass would spill 20 of
// them (1024^2 x 256, 20 steps: 2640 -> 2210 us), its dual passes 3 (2340 ->
// 2240 us).  Row offsets are then added at use, the objective's sums live in
// LDS and the partial steps have one code path.  Depth 3 has the registers, and
// there each of these costs (512^2 x 128, 20 steps: 2183 us without, 2270 with).
__host__ __device__ constexpr bool tv_lean(int LV) { return LV > 3; }
// Form of a pass: the pipeline above, or (SEQ) step l at plane a1 - l, every step
// behind a barrier of its own, planes prefetched two ahead, FIRST known when
// compiled.  A pass of one step or none, or over few planes, does not fill the
// pipeline: its planes take less than their loads, and idle phases and the plane that
// steps 2 and 3 wait are what it pays.  Prox of one step at 512^2 x 128 in 3D 214 ->
// 112 us (with the z cut of such passes), none 135 -> 60; plane groups of one plane at
// 768^2 x 50, 10 steps, 2.58 -> 1.95 ms; 64^2 x 8 in 2D, 10 steps, 24 -> 19 us.
enum TvForm { TV_PIPE, TV_SEQ, TV_SEQ_FIRST };
// Slots of s_py per step.  From depth 3 on an iteration of the pipeline has two
// barriers, so a row is read long before it is replaced and one slot would do, which
// depth 4 takes (the sums' room); with one barrier the slots alternate.
__host__ __device__ constexpr int tv_py_slots(int LV, TvForm F) { return F == TV_PIPE && tv_lean(LV) ? 1 : 2; }
// Slots of the v ring: back to the last step's plane, on the final pass to the
// output plane.
template <int LV, bool FINAL, bool SEQ>
__host__ __device__ constexpr int tv_ring() { return FINAL ? (SEQ ? LV : tv_delay(LV)) + 1 : tv_delay(LV); }

// Bound on a wave's wait for another segment to publish a row-store index
// (about 2^20 * 128 clocks; the publisher needs a few hundred).
constexpr int kStoreSpinLimit = 1 << 20;

template <int H, int LV, int Q, TvForm F, bool EDGE, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
__device__ __forceinline__ void tv_pass_body(const TvPassArgs& A, int bx, int by, int zb, int ze, int blk,
                                             float (*s_py)[tv_py_slots(LV, F)][kTvWaves][64], float (*s_ut)[2][kTvWaves][64],
                                             TvVec<Q>* s_v, float (*s_x)[kTvWaves][64], double (*s_red)[kTvWaves],
                                             float* s_fin, double* s_sum) {
  constexpr int NW = kTvWaves, NT = NW * 64, RY = NW * Q;
  constexpr int IX = kTvRX - 2 * H, IY = RY - 2 * H;  // interior (stored) extent
  constexpr int PYM = tv_py_slots(LV, F) - 1;
  constexpr bool SEQ = F != TV_PIPE, FIRST = F == TV_SEQ_FIRST;
  constexpr bool LEAN = tv_lean(LV);
  const float* __restrict__ v =
      uniform_ptr((A.v ? A.v : pick3(A.vol[0], A.vol[1], A.vol[2], A.st->prev)) + A.zoff_v);
  float* __restrict__ xo = uniform_ptr((A.x ? A.x : pick3(A.vol[0], A.vol[1], A.vol[2], A.st->next)) + A.zoff_x);
  const int nx = A.nx, ny = A.ny, nz = A.nz;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // dual buffers of this pass: with a warm-started dual the sets alternate
  // from one outer iteration to the next when a prox has an odd number of passes
  const bool flip = A.flip_npass > 0 && A.st != nullptr && (((A.st->it - 1) * A.flip_npass) & 1);
  const float* pin[3];
  float* pout[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    pin[k] = uniform_ptr(flip ? const_cast<const float*>(A.pout[k]) : A.pin[k]);
    pout[k] = uniform_ptr(flip ? const_cast<float*>(A.pin[k]) : A.pout[k]);
  }
  constexpr bool bf = BF;   // dual buffers in bfloat16
  const bool first = A.first != 0;   // the incoming dual is zero: read as zeros through empty descriptors
  const int x = bx * IX - H + lane;
  const int ybase = by * IY - H + wv * Q;
  const bool inx = !EDGE || (x >= 0 && x < nx);
  const bool xlo = !EDGE || x > 0, xhi = !EDGE || x + 1 < nx;
  const bool ix_store = inx && lane >= H && lane < kTvRX - H;
  const size_t sz = (size_t)nx * ny;
  const int L = A.levels;

  const int M = TV2 ? 0 : L + 1;
  const int zs = max(0, zb - M), zl = min(nz, ze + M);
  const float tau = A.tau, cc = A.c;

  bool ylo[Q], yhi[Q], ys[Q];
  // In-plane byte offsets: one of the lane and one of the wave's row.  kTvOff:
  // outside the volume (loads), the stored interior (stores).
  const unsigned xoff = inx ? (unsigned)x * 4u : kTvOff, xoffs = ix_store ? (unsigned)x * 4u : kTvOff;
  unsigned rowl[Q], rows[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int y = ybase + q;
    const bool iny = !EDGE || (y >= 0 && y < ny);
    ylo[q] = !EDGE || y > 0;
    yhi[q] = !EDGE || y + 1 < ny;
    const int r = wv * Q + q;
    ys[q] = ix_store && iny && r >= H && r < RY - H;
    rowl[q] = iny ? (unsigned)(y * nx) * 4u : kTvOff;
    rows[q] = iny && r >= H && r < RY - H ? rowl[q] : kTvOff;
  }
  // (lean: the empty statement keeps the sums out of registers that live through the march)
  auto load_off = [&](int q) __attribute__((always_inline)) {
    unsigned r = rowl[q];
    if constexpr (LEAN) asm volatile("" : "+s"(r));
    return r + xoff;
  };
  auto store_off = [&](int q) __attribute__((always_inline)) {
    unsigned r = rows[q];
    if constexpr (LEAN) asm volatile("" : "+s"(r));
    return r + xoffs;
  };
  // per fused step: previous plane's dual (3) and primal (1)
  float Pp[LV][Q][3], Up[LV][Q];
#pragma unroll
  for (int l = 0; l < LV; ++l)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      Pp[l][q][0] = Pp[l][q][1] = Pp[l][q][2] = 0.f;
      Up[l][q] = 0.f;
    }
  // Final-pass state kept in thread-private LDS rather than registers (the
  // final pass holds H fused steps in a tile of halo H + 1 and would spill):
  // the previous output plane's p_z (PzF) and x (Xp).
  auto PzF = [&](int q) __attribute__((always_inline)) -> float& { return s_fin[q * NT + threadIdx.x]; };
  auto Xp = [&](int q) __attribute__((always_inline)) -> float& { return s_fin[(Q + q) * NT + threadIdx.x]; };
  const bool obj = FINAL && A.psum != nullptr;
  if constexpr (FINAL) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      PzF(q) = 0.f;
      Xp(q) = 0.f;
    }
  }
  // ||x||_1 and TV(x) of the thread's voxels (objective pieces), and what their
  // additions dropped
  constexpr bool SUMS = FINAL && LEAN, LOS = SUMS && !SEQ;   // (the second s_py slots of SEQ take the room)
  double r_sum[2];
  float r_lo[2];
  double& x_sum = *(SUMS ? s_sum + threadIdx.x : r_sum);
  double& tv_sum = *(SUMS ? s_sum + NT + threadIdx.x : r_sum + 1);
  float* const s_lo = reinterpret_cast<float*>(s_sum + 2 * NT);
  float& x_lo = *(LOS ? s_lo + threadIdx.x : r_lo);
  float& tv_lo = *(LOS ? s_lo + NT + threadIdx.x : r_lo + 1);
  x_sum = tv_sum = 0.0;
  x_lo = tv_lo = 0.f;
  // terms of the plane held in Xp; xn: the next plane (hz: it exists), slot:
  // the LDS slot holding the first row of every wave of the Xp plane
  auto accumulate = [&](const float* xn, bool hz, int slot) __attribute__((always_inline)) {
    float xq[Q], tq[Q], any = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float x0 = Xp(q);
      const float xr = dpp_from_right(x0);
      const float xu = (q < Q - 1) ? Xp(q + 1) : s_x[slot][wv < NW - 1 ? wv + 1 : wv][lane];
      const float gx = xhi ? xr - x0 : 0.f;
      const float gy = yhi[q] ? xu - x0 : 0.f;
      const float gz = (hz && !TV2) ? xn[q] - x0 : 0.f;
      // per-voxel norm in FP32 (the hardware square root, within 1 ulp, not
      // the correctly rounded sequence), running sums in FP64
      const float t = __builtin_amdgcn_sqrtf(fmaf(gx, gx, fmaf(gy, gy, gz * gz)));
      xq[q] = ys[q] ? fabsf(x0) : 0.f;   // ||x||_1
      tq[q] = ys[q] ? t : 0.f;
      any += xq[q] + tq[q];
    }
    if (__ballot(any != 0.f) == 0) return;   // nothing but zeros in the wave's rows (most planes of a sparse volume)
    // (a few FP32 terms add up exactly in FP64 unless they span 2^27)
    double xp = 0.0, tp = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      xp += (double)xq[q];
      tp += (double)tq[q];
    }
    double xs = x_sum, ts = tv_sum;
    float xl = x_lo, tl = tv_lo;
    add_exact(xs, xl, xp);
    add_exact(ts, tl, tp);
    x_sum = xs;
    tv_sum = ts;
    x_lo = xl;
    tv_lo = tl;
  };

  // Input planes are prefetched one ahead (a plane of the pipeline takes about 4 us),
  // or two (SEQ).  v of recent planes lives in a thread-private LDS ring (slot = plane mod NS).
  struct InPlane {
    float v[Q];
    float p[Q][3];
    float pp[Q][3];   // FGP: p_prev of the plane
  };
  auto load_plane = [&](InPlane& P, int a) __attribute__((always_inline)) {
    unsigned off[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) off[q] = load_off(q);
    const __amdgpu_buffer_rsrc_t rv = plane_rsrc(v, a, sz);
#pragma unroll
    for (int q = 0; q < Q; ++q) P.v[q] = buf_ld(rv, off[q]);
    if constexpr (FIRST) return;
    const __amdgpu_buffer_rsrc_t r0 = dual_rsrc(pin[0], a, sz, bf, first);
    const __amdgpu_buffer_rsrc_t r1 = dual_rsrc(pin[1], a, sz, bf, first);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      P.p[q][0] = dual_ld(r0, off[q], bf);
      P.p[q][1] = dual_ld(r1, off[q], bf);
    }
    if constexpr (!TV2) {
      const __amdgpu_buffer_rsrc_t r2 = dual_rsrc(pin[2], a, sz, bf, first);
#pragma unroll
      for (int q = 0; q < Q; ++q) P.p[q][2] = dual_ld(r2, off[q], bf);
    }
    if constexpr (FGP) {
      const __amdgpu_buffer_rsrc_t s0 = dual_rsrc(A.pin2[0], a, sz, bf, first);
      const __amdgpu_buffer_rsrc_t s1 = dual_rsrc(A.pin2[1], a, sz, bf, first);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        P.pp[q][0] = dual_ld(s0, off[q], bf);
        P.pp[q][1] = dual_ld(s1, off[q], bf);
        P.pp[q][2] = 0.f;
      }
      if constexpr (!TV2) {
        const __amdgpu_buffer_rsrc_t s2 = dual_rsrc(A.pin2[2], a, sz, bf, first);
#pragma unroll
        for (int q = 0; q < Q; ++q) P.pp[q][2] = dual_ld(s2, off[q], bf);
      }
    }
  };
  constexpr int NS = tv_ring<LV, FINAL, SEQ>();
  auto vring = [&](int a) __attribute__((always_inline)) -> TvVec<Q>& { return s_v[(a % NS) * NT + threadIdx.x]; };

  // Arrival of the previous dual c3 at plane a for fused step l: u(a), then
  // the dual step at plane a - 1 (which needs u(a) for its z-difference) into
  // c3.  arrive_pre publishes the row the wave above needs and fetches v;
  // a barrier separates the two halves.
  auto arrive_pre = [&](int l, int a, int par, const float (&c3)[Q][3], float (&un)[Q]) __attribute__((always_inline)) {
    const TvVec<Q> vq = vring(a);  // thread-private: read before the barrier
#pragma unroll
    for (int q = 0; q < Q; ++q) un[q] = vq[q];
    s_py[l][par & PYM][wv][lane] = c3[Q - 1][1];
  };
  auto arrive_post = [&](int l, bool start, int par, float (&c3)[Q][3], float (&un)[Q]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float pxm = dpp_from_left(c3[q][0]);
      const float pym = (q > 0) ? c3[q - 1][1] : s_py[l][par & PYM][wv > 0 ? wv - 1 : 0][lane];
      float d = (xhi ? c3[q][0] : 0.f) - (xlo ? pxm : 0.f);
      d += (yhi[q] ? c3[q][1] : 0.f) - (ylo[q] ? pym : 0.f);
      if constexpr (!TV2) d += c3[q][2] - Pp[l][q][2];
      un[q] = fmaf(tau, d, un[q]);
    }
    if (!start) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float u0 = Up[l][q];
        const float uxp = dpp_from_right(u0);
        const float uyp = (q < Q - 1) ? Up[l][q + 1] : s_ut[l][par ^ 1][wv < NW - 1 ? wv + 1 : wv][lane];
        const float gx = xhi ? uxp - u0 : 0.f;
        const float gy = yhi[q] ? uyp - u0 : 0.f;
        const float gz = un[q] - u0;       // plane a exists
        const float qx = fmaf(cc, gx, Pp[l][q][0]);
        const float qy = fmaf(cc, gy, Pp[l][q][1]);
        const float qz = TV2 ? 0.f : fmaf(cc, gz, Pp[l][q][2]);
        const float n2 = fmaf(qx, qx, fmaf(qy, qy, qz * qz));
        const float sc = fminf(1.f, __frsqrt_rn(n2));   // 1 / max(1, |q|)
        Pp[l][q][0] = c3[q][0];
        Pp[l][q][1] = c3[q][1];
        Pp[l][q][2] = c3[q][2];
        c3[q][0] = qx * sc;
        c3[q][1] = qy * sc;
        c3[q][2] = qz * sc;
      }
      // Up is read by the neighbours above (q+1) before it is replaced
#pragma unroll
      for (int q = 0; q < Q; ++q) Up[l][q] = un[q];
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        Pp[l][q][0] = c3[q][0];
        Pp[l][q][1] = c3[q][1];
        Pp[l][q][2] = c3[q][2];
        Up[l][q] = un[q];
      }
    }
    s_ut[l][par][wv][lane] = un[0];
  };
  // Flush of fused step l: dual step at the last plane zl - 1 (no plane above).
  auto flush = [&](int l, int par, float (&c3)[Q][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float u0 = Up[l][q];
      const float uxp = dpp_from_right(u0);
      const float uyp = (q < Q - 1) ? Up[l][q + 1] : s_ut[l][par ^ 1][wv < NW - 1 ? wv + 1 : wv][lane];
      const float gx = xhi ? uxp - u0 : 0.f;
      const float gy = yhi[q] ? uyp - u0 : 0.f;
      const float qx = fmaf(cc, gx, Pp[l][q][0]);
      const float qy = fmaf(cc, gy, Pp[l][q][1]);
      const float qz = TV2 ? 0.f : Pp[l][q][2];
      const float n2 = fmaf(qx, qx, fmaf(qy, qy, qz * qz));
      const float sc = fminf(1.f, __frsqrt_rn(n2));
      c3[q][0] = qx * sc;
      c3[q][1] = qy * sc;
      c3[q][2] = qz * sc;
    }
  };
  // Output stage: the dual of the last fused step at plane m (stored), or on
  // the final pass the primal recovery, soft threshold, store and flags.
  // The stores are issued whatever m is (through empty descriptors where the
  // plane is not this block's): were they skipped by a branch, the wait for the
  // prefetched plane, whose loads are older, would have to allow for none of
  // them in between and so wait for the stores as well.
  auto store3 = [&](float* const* dst, int m, const float (&c3)[Q][3], bool on) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t o0 = dual_rsrc(dst[0], m, sz, bf, !on);
    const __amdgpu_buffer_rsrc_t o1 = dual_rsrc(dst[1], m, sz, bf, !on);
    unsigned offs[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) offs[q] = store_off(q);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      dual_st(o0, offs[q], c3[q][0], bf);
      dual_st(o1, offs[q], c3[q][1], bf);
    }
    if constexpr (!TV2) {
      const __amdgpu_buffer_rsrc_t o2 = dual_rsrc(dst[2], m, sz, bf, !on);
#pragma unroll
      for (int q = 0; q < Q; ++q) dual_st(o2, offs[q], c3[q][2], bf);
    }
  };
  // FGP: p_prev of the plane that arrived last (the next plane to be output)
  float PPv[Q][3];
#pragma unroll
  for (int q = 0; q < Q; ++q) PPv[q][0] = PPv[q][1] = PPv[q][2] = 0.f;
  auto store_dual = [&](int m, const float (&c3)[Q][3], bool on) __attribute__((always_inline)) {
    if constexpr (FGP) {
      // c3 is p at plane m; the next pass steps at r_next = p + w (p - p_prev)
      const float w = A.fgp_w;
      float rn[Q][3];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int k = 0; k < 3; ++k) rn[q][k] = fmaf(w, c3[q][k] - PPv[q][k], c3[q][k]);
      store3(pout, m, rn, on);
      store3(A.pout2, m, c3, on);
    } else {
      store3(pout, m, c3, on);
    }
  };
  // Row-compressed store of x_{k+1} (A.rs.on): this wave's segments of rows
  // ybase .. ybase + Q - 1 of plane m; bit q of nzm: segment q holds a
  // non-zero value.  Lane q claims row q's slot (-1 -> -2) when it is still
  // absent; the claimed rows take consecutive pool rows with one counter
  // update and their indices are published; a row found claimed by another
  // segment is waited for (its claimer depends on nothing, so the wait ends;
  // a bound on it reports an overflow instead).  Slot -3: the pool ran out.
  // Pool rows not in use are zero (zeroed at the start and when a store is
  // recycled), so a segment writes only its values and no ordering beyond the
  // slots' atomics is needed; every occupied row takes exactly one pool row.
  auto store_rows = [&](int m, const float (&xs)[Q], unsigned nzm, bool zstore) __attribute__((always_inline)) {
    const int k = A.st->scur ^ 1;
    float* pool = k == 0 ? A.rs.pool[0] : A.rs.pool[1];
    const bool mine = lane < Q && ((nzm >> lane) & 1u);
    int32_t* tab = (k == 0 ? A.rs.slot[0] : A.rs.slot[1]) + (size_t)m * ny + (mine ? ybase + lane : 0);
    int idx = -1;
    if (mine) idx = __hip_atomic_load(tab, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (mine && idx == -1) {
      idx = atomicCAS(tab, -1, -2);
      idx = idx == -1 ? -4 : idx;          // -4: this lane won the claim
    }
    const uint64_t wm = __ballot(mine && idx == -4);
    if (wm != 0) {
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&A.rs.count[k], (uint32_t)__popcll(wm));
      base = __builtin_amdgcn_readfirstlane(base);
      if (mine && idx == -4) {
        const uint32_t sn = base + (uint32_t)__popcll(wm & ((1ull << lane) - 1ull));
        idx = sn < A.rs.cap ? (int)sn : -3;
        if (idx < 0) atomicOr(A.rs.overflow, 1u);
        __hip_atomic_store(tab, idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    for (int spin = 0; __ballot(mine && idx == -2) != 0; ++spin) {
      if (spin >= kStoreSpinLimit) {
        if (mine && idx == -2) {
          atomicOr(A.rs.overflow, 2u);
          idx = -3;
        }
        break;
      }
      __builtin_amdgcn_s_sleep(2);
      if (mine && idx == -2) idx = __hip_atomic_load(tab, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (!((nzm >> q) & 1u)) continue;
      const int r = __builtin_amdgcn_readlane(idx, q);
      if (r >= 0 && zstore && ys[q]) pool[(size_t)r * nx + x] = xs[q];
    }
  };
  auto output = [&](int m, int par, float (&c3)[Q][3]) __attribute__((always_inline)) {
    const bool zstore = m >= zb && m < ze;
    if constexpr (!FINAL) {
      store_dual(m, c3, zstore);
    } else {
      if (A.keep_dual) store_dual(m, c3, zstore);
      const TvVec<Q> vm = vring(m);  // thread-private: read before the barrier
      // no step, dual zero: nothing to exchange but the objective's rows
      const bool still = FIRST && L == 0;
      if (!still) s_py[LV][par & PYM][wv][lane] = c3[Q - 1][1];
      if (!still || obj) __syncthreads();
      const __amdgpu_buffer_rsrc_t rx = dual_rsrc(xo, m, sz, false, !zstore);
      float xs[Q];
      unsigned nzm = 0;   // row-compressed store: segments holding a non-zero
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float u = vm[q];
        if (tau != 0.f) {
          const float pxm = dpp_from_left(c3[q][0]);
          const float pym = (q > 0) ? c3[q - 1][1] : (still ? 0.f : s_py[LV][par & PYM][wv > 0 ? wv - 1 : 0][lane]);
          float d = (xhi ? c3[q][0] : 0.f) - (xlo ? pxm : 0.f);
          d += (yhi[q] ? c3[q][1] : 0.f) - (ylo[q] ? pym : 0.f);
          if constexpr (!TV2) d += c3[q][2] - PzF(q);
          u = fmaf(tau, d, u);
        }
        if constexpr (!TV2) PzF(q) = c3[q][2];
        float xv;
        if (A.nonneg) {
          xv = fmaxf(u - A.thr, 0.f);
        } else {
          xv = copysignf(fmaxf(fabsf(u) - A.thr, 0.f), u);
        }
        xs[q] = xv;
        const bool st = zstore && ys[q];
        const bool nzr = __ballot(st && xv != 0.f) != 0;   // this wave's segment of the row holds a non-zero
        if constexpr (SP) {
          nzm |= nzr ? 1u << q : 0u;   // stored below, the wave's rows together
        } else {
          buf_st(rx, store_off(q), xv);
        }
        if (A.rowflag != nullptr) {
          if (nzr && lane == 0) {
            A.rowflag[(size_t)m * ny + ybase + q] = 1;
            A.planeflag[m] = 1;
          }
        }
      }
      if constexpr (SP) {
        if (nzm != 0) store_rows(m, xs, nzm, zstore);
      }
      if (obj) {
        // plane m - 1 is complete now; its first rows went to slot par ^ 1
        if (m - 1 >= zb && m - 1 < ze) accumulate(xs, true, par ^ 1);
        s_x[par][wv][lane] = xs[0];  // read after the next output's barrier
#pragma unroll
        for (int q = 0; q < Q; ++q) Xp(q) = xs[q];
      }
    }
  };

  float C[Q][3];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int k = 0; k < 3; ++k) C[q][k] = 0.f;
  const int delay = SEQ ? L : tv_delay(L);   // the output plane is a1 - delay
  const int nsteps = zl - zs + delay;        // the last output leaves at s = nsteps - 1
  InPlane P;
  if constexpr (SEQ) {
    auto arrive = [&](int l, int a, int par) __attribute__((always_inline)) {
      float un[Q];
      arrive_pre(l, a, par, C, un);
      __syncthreads();
      arrive_post(l, a == zs, par, C, un);
    };
    auto step = [&](InPlane& P, int s) __attribute__((always_inline)) {
      const int par = s & 1, a1 = zs + s;
      float ppa[Q][3];   // FGP: p_prev of plane a1 (one step: output of a1 comes at the next arrival)
      TvVec<Q> vq;
#pragma unroll
      for (int q = 0; q < Q; ++q) vq[q] = vcopy(P.v[q]);
      vring(a1) = vq;
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          C[q][k] = FIRST || (TV2 && k == 2) ? 0.f : dual_val(P.p[q][k], bf);
          if constexpr (FGP) ppa[q][k] = FIRST || (TV2 && k == 2) ? 0.f : dual_val(P.pp[q][k], bf);
        }
      if (a1 + 2 < zl) load_plane(P, a1 + 2);
#pragma unroll
      for (int l = 0; l < LV; ++l) {
        if (l >= L || a1 - l < zs) break;   // this and the later steps are idle
        arrive(l, a1 - l, par);
      }
      if (a1 - L >= zs) output(a1 - L, par, C);
      if constexpr (FGP) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int k = 0; k < 3; ++k) PPv[q][k] = ppa[q][k];
      }
    };
    InPlane R;
    load_plane(P, zs);
    if (zs + 1 < zl) load_plane(R, zs + 1);
    for (int s = 0; s < zl - zs; s += 2) {   // (two register sets in turn)
      step(P, s);
      if (s + 1 < zl - zs) step(R, s + 1);
    }
    // no plane arrives any more: step l flushes at s = zl - zs + l
    for (int s = zl - zs; s < nsteps; ++s) {
      const int par = s & 1, a1 = zs + s;
#pragma unroll
      for (int l = 0; l < LV; ++l) {
        const int a = a1 - l;
        if (l >= L || a < zs) break;
        if (a > zl) continue;
        if (a == zl) {
          __syncthreads();
          flush(l, par, C);
        } else {
          arrive(l, a, par);
        }
      }
      if (a1 - L >= zs) output(a1 - L, par, C);
    }
  } else {
    // One plane of the pipeline: plane a1 = zs + s arrives (none past zl).  Steps 0
    // and 2 run side by side between two barriers, then steps 1 and 3: step 2
    // takes what step 1 left in the iteration before (its dual waits in D), so
    // it sits one plane further back, step l at plane a1 - l - (l > 1).  Two
    // independent steps per barrier fill the latencies of each other's exchange.
    // A step is idle before its first plane, at plane zl it flushes, then idles
    // again.  EACH = false: the steady part, where all LV steps are arrivals.
    float D[Q][3];   // dual after steps 1 / 2 / 3 (C: after steps 0 / 1)
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int k = 0; k < 3; ++k) D[q][k] = 0.f;
    auto iterate = [&](auto each, int s) __attribute__((always_inline)) {
      constexpr bool EACH = decltype(each)::value;
      const int par = s & 1;
      const int a1 = zs + s;
      float ppa[Q][3];   // FGP: p_prev of plane a1 (one step: output of a1 comes at the next arrival)
      if (!EACH || a1 < zl) {
        TvVec<Q> vq;
#pragma unroll
        for (int q = 0; q < Q; ++q) vq[q] = vcopy(P.v[q]);
        vring(a1) = vq;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          C[q][0] = dual_val(P.p[q][0], bf);
          C[q][1] = dual_val(P.p[q][1], bf);
          C[q][2] = TV2 ? 0.f : dual_val(P.p[q][2], bf);
          if constexpr (FGP) {
#pragma unroll
            for (int k = 0; k < 3; ++k) ppa[q][k] = dual_val(P.pp[q][k], bf);
          }
        }
        if (a1 + 1 < zl) load_plane(P, a1 + 1);
      } else if constexpr (FGP) {
#pragma unroll
        for (int q = 0; q < Q; ++q) ppa[q][0] = ppa[q][1] = ppa[q][2] = 0.f;
      }
      auto arrives = [&](int l, int a) __attribute__((always_inline)) { return !EACH || (l < L && a >= zs && a < zl); };
      auto flushes = [&](int l, int a) __attribute__((always_inline)) { return EACH && l < L && a == zl; };
      // one phase: step l on x at plane a, and step m (if the kernel has it) on y at plane b
      auto phase = [&](auto lc, auto mc, int a, float (&x)[Q][3], int b, float (&y)[Q][3]) __attribute__((always_inline)) {
        constexpr int l = decltype(lc)::value, m = decltype(mc)::value;
        float ul[Q], um[Q];
        if (arrives(l, a)) arrive_pre(l, a, par, x, ul);
        if constexpr (m < LV)
          if (arrives(m, b)) arrive_pre(m, b, par, y, um);
        __syncthreads();
        if (arrives(l, a)) arrive_post(l, EACH && a == zs, par, x, ul);
        else if (flushes(l, a)) flush(l, par, x);
        if constexpr (m < LV) {
          if (arrives(m, b)) arrive_post(m, EACH && b == zs, par, y, um);
          else if (flushes(m, b)) flush(m, par, y);
        }
      };
      using std::integral_constant;
      phase(integral_constant<int, 0>{}, integral_constant<int, 2>{}, a1, C, a1 - 3, D);
      const int m = a1 - delay;
      const bool outs = !EACH || (m >= zs && m < zl);
      // the output of C or D, chosen value by value (two branches that differ in
      // the array alone would be merged and keep both arrays in memory)
      auto output_of = [&](bool d) __attribute__((always_inline)) {
        float O[Q][3];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int k = 0; k < 3; ++k) O[q][k] = d ? D[q][k] : C[q][k];
        output(m, par, O);
      };
      if (EACH ? outs && (L < 2 || L == 3) : LV == 3) output_of(EACH ? L == 3 : true);
      if (!EACH || L > 1) {
        if constexpr (LV == 2) phase(integral_constant<int, 1>{}, integral_constant<int, LV>{}, a1 - 1, C, 0, D);
        else phase(integral_constant<int, 1>{}, integral_constant<int, 3>{}, a1 - 1, C, a1 - 4, D);
        if (EACH ? outs && (L == 2 || L == 4) : LV != 3) output_of(EACH ? L == 4 : LV == 4);
        if constexpr (LV > 2) {
          // the dual after step 1 waits for step 2
#pragma unroll
          for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int k = 0; k < 3; ++k) D[q][k] = C[q][k];
        }
      } else if constexpr (LEAN) {
        __syncthreads();   // the iteration's second barrier (s_py)
      }
      if constexpr (FGP) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int k = 0; k < 3; ++k) PPv[q][k] = ppa[q][k];
      }
      // the next plane's copies, and the waits for its loads, stay behind this
      // plane's arithmetic
      __builtin_amdgcn_sched_barrier(0);
    };
    load_plane(P, zs);
    // steady part: every step has its first plane behind it, a1 < zl
    const int s0 = tv_delay(LV) + 1;
    const int s1 = L == LV && zl - zs > s0 ? zl - zs : 0;
    if constexpr (LEAN) {
      for (int s = 0; s < nsteps; ++s) {
        if (s == s0) {
          for (; s + 1 < s1; s += 2) {
            iterate(std::false_type{}, s);
            iterate(std::false_type{}, s + 1);
          }
        }
        iterate(std::true_type{}, s);
      }
    } else {
      int s = 0;
      if (s1 > 0) {
        for (; s < s0; ++s) iterate(std::true_type{}, s);
        for (; s + 1 < s1; s += 2) {
          iterate(std::false_type{}, s);
          iterate(std::false_type{}, s + 1);
        }
      }
      for (; s < nsteps; ++s) iterate(std::true_type{}, s);
    }
  }
  if constexpr (FINAL) {
    if (obj) {
      if (ze == nz || TV2) {
        // the last plane of the volume: no plane above it (its z-difference is
        // 0); in 2D the last plane of every chunk, which has no z margin
        __syncthreads();
        accumulate(nullptr, false, (nsteps - 1) & 1);
      }
      double acc[2] = {x_sum, tv_sum}, lo[2] = {(double)x_lo, (double)tv_lo};
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
          const double oh = __shfl_xor(acc[k], off, 64);
          lo[k] += __shfl_xor(lo[k], off, 64);
          add_exact(acc[k], lo[k], oh);
        }
        if (lane == 0) {
          s_red[2 * k][wv] = acc[k];
          s_red[2 * k + 1][wv] = lo[k];
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          double s = 0.0, l = 0.0;
          for (int w = 0; w < NW; ++w) {
            l += s_red[2 * k + 1][w];
            add_exact(s, l, s_red[2 * k][w]);
          }
          double* dst = (k == 0 ? A.psum : A.ptv) + 2 * (size_t)blk;
          dst[0] = s;
          dst[1] = l;
        }
      }
    }
  }
}

// HT: tile halo, LV: fused-step register slots.  Dual passes use HT = LV = H;
// the final pass HT = H + 1, LV = H.
template <int HT, int LV, int Q, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
__device__ __forceinline__ void tv_pass_entry(const TvPassArgs& A, int bx, int by, int zb, int ze, int blk) {
  __shared__ float s_py[LV + 1][tv_py_slots(LV, SEQ ? TV_SEQ : TV_PIPE)][kTvWaves][64];  // bottom-row p_y per wave, per step (+ final)
  __shared__ float s_ut[LV][2][kTvWaves][64];      // top-row u per wave, per step, parity
  __shared__ TvVec<Q> s_v[tv_ring<LV, FINAL, SEQ>() * kTvWaves * 64];  // v ring, thread-private
  __shared__ float s_x[FINAL ? 2 : 1][kTvWaves][64];     // final pass: first-row x per wave, parity
  __shared__ double s_red[4][kTvWaves];            // final pass: per-wave sums
  __shared__ float s_fin[FINAL ? 2 * Q * kTvWaves * 64 : 1];    // final pass: PzF, Xp (thread-private)
  __shared__ double s_sum[FINAL && tv_lean(LV) ? (SEQ ? 2 : 3) * kTvWaves * 64 : 1];   // final pass: sums (thread-private)
  // the stop flag read once per wave (a wave-uniform branch)
  if (A.st != nullptr && __builtin_amdgcn_readfirstlane(A.st->done)) return;
  constexpr int RY = kTvWaves * Q, IX = kTvRX - 2 * HT, IY = RY - 2 * HT;
  const int x0 = bx * IX - HT, y0 = by * IY - HT;
  // interior tile: every point of the region and its +-1 neighbours lie inside
  const bool interior = x0 >= 1 && x0 + kTvRX <= A.nx - 1 && y0 >= 1 && y0 + RY <= A.ny - 1;
  auto* sx = reinterpret_cast<float (*)[kTvWaves][64]>(&s_x[0][0][0]);
#define RIHVR_TV_BODY(F, E) \
  tv_pass_body<HT, LV, Q, F, E, FINAL, TV2, FGP, BF, SP>(A, bx, by, zb, ze, blk, s_py, s_ut, s_v, sx, s_red, s_fin, s_sum)
  if constexpr (SEQ) {
    if (A.first) {
      if (interior) RIHVR_TV_BODY(TV_SEQ_FIRST, false);
      else RIHVR_TV_BODY(TV_SEQ_FIRST, true);
    } else {
      if (interior) RIHVR_TV_BODY(TV_SEQ, false);
      else RIHVR_TV_BODY(TV_SEQ, true);
    }
  } else {
    if (interior) RIHVR_TV_BODY(TV_PIPE, false);
    else RIHVR_TV_BODY(TV_PIPE, true);
  }
#undef RIHVR_TV_BODY
}

// The second launch-bounds argument is the minimum number of waves per SIMD
// the register allocation must allow: 12-wave blocks need 3 (<= 170 VGPRs,
// one block per CU), which every fusion depth fits.
constexpr int kTvWavesPerSimd = (kTvWaves + 3) / 4;

// Work of block t of a pass (t < A.nblocks): the first nfull tiles (raster
// order) times their z chunks of zchunk planes, tile-fastest; then the other
// tiles times their chunks of zchunk2 planes.
struct TvWork {
  int bx, by, zb, ze;
};
__device__ __forceinline__ TvWork tv_work(const TvPassArgs& A, uint32_t t) {
  const uint32_t n1 = (uint32_t)A.nfull * (uint32_t)((A.nz + A.zchunk - 1) / A.zchunk);
  uint32_t tile, zb, zc;
  if (t < n1) {
    tile = t % A.nfull;
    zc = A.zchunk;
    zb = (t / A.nfull) * zc;
  } else {
    const uint32_t r = (uint32_t)(A.gx * A.gy - A.nfull), u = t - n1;
    tile = A.nfull + u % r;
    zc = A.zchunk2;
    zb = (u / r) * zc;
  }
  TvWork w;
  w.bx = (int)(tile % A.gx);
  w.by = (int)(tile / A.gx);
  w.zb = (int)zb;
  w.ze = min(A.nz, (int)(zb + zc));
  return w;
}

// The first part of the grid (whole rounds of tiles) takes the XCD-contiguous
// order; the thin chunks of the split tiles, dispatched last, keep the
// hardware order so that they spread over every XCD.
template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP, int Q = kTvQ>
__global__ void __launch_bounds__(kTvWaves * 64, kTvWavesPerSimd) k_tv_pass(TvPassArgs A) {
  const uint32_t hw = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const uint32_t n1 = (uint32_t)A.nfull * (uint32_t)((A.nz + A.zchunk - 1) / A.zchunk);
  const uint32_t t = hw < n1 ? xcd_tile(hw, n1) : hw;
  const TvWork w = tv_work(A, t);
  tv_pass_entry<FINAL ? H + 1 : H, FGP ? 1 : H, Q, SEQ, FINAL, TV2, FGP, BF, SP>(A, w.bx, w.by, w.zb, w.ze, (int)t);
}

// Work item b of a batched launch: the frame f with offs[f] <= b < offs[f+1]
// and block b - offs[f] of that frame's pass.
template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
__device__ __forceinline__ void tv_batch_item(const TvPassArgs* __restrict__ args, const BatchMap& map, uint32_t b) {
  int lo = 0, hi = map.n;  // largest f with offs[f] <= b
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (map.offs[mid] <= b) lo = mid;
    else hi = mid;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);  // uniform: the frame's arguments come in as scalar loads
  // read in place (scalar loads when used) rather than copied: a copy of the
  // whole struct held in scalar registers for the kernel's lifetime spills
  const TvPassArgs& A = args[lo];
  const int lb = (int)(b - (uint32_t)__builtin_amdgcn_readfirstlane(map.offs[lo]));
  const TvWork w = tv_work(A, (uint32_t)lb);
  tv_pass_entry<FINAL ? H + 1 : H, FGP ? 1 : H, kTvQ, SEQ, FINAL, TV2, FGP, BF, SP>(A, w.bx, w.by, w.zb, w.ze, lb);
}

template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
__global__ void __launch_bounds__(kTvWaves * 64, kTvWavesPerSimd) k_tv_pass_b(const TvPassArgs* __restrict__ args,
                                                                                  BatchMap map) {
  tv_batch_item<H, SEQ, FINAL, TV2, FGP, BF, SP>(args, map, xcd_tile(blockIdx.x, gridDim.x));
}

// Persistent form of the batched pass: a grid of about one block per compute
// unit takes the launch's work items (every frame's blocks end to end, as
// above) from a device queue instead of running one item per block.  The items
// are cut into one contiguous range per XCD, each with a claim counter; a
// block claims items one at a time with an atomic add, from its own XCD's
// range first (neighbouring tiles share that XCD's L2), then from the other
// ranges in turn, so that the blocks that run out of work early take over the
// tail.  Items are independent and a block runs one whole item between two
// barriers, so the results do not depend on which block ran which item.  The
// last block out resets the counters: the next launch, a graph replay
// included, finds them at zero.
// The claim takes no branch on the thread index: every thread adds to the
// counter (thread 0 one, the others zero) and to the LDS word (thread 0 its
// claim, the others zero).  A branch on thread 0 here, next to the final
// pass's own thread-0 epilogue at the end of an item, lets the compiler thread
// the two across the loop's back edge and turn the item loop into an
// exec-masked loop with the barriers inside, which waves leave after
// different numbers of trips.
template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
__global__ void __launch_bounds__(kTvWaves * 64, kTvWavesPerSimd) k_tv_pass_q(const TvPassArgs* __restrict__ args,
                                                                                  BatchMap map) {
  __shared__ uint32_t s_item;
  const uint32_t n = __builtin_amdgcn_readfirstlane(map.offs[map.n]);
  const uint32_t q = n / kXcds, r = n % kXcds, home = blockIdx.x % kXcds;
  const uint32_t one = threadIdx.x == 0 ? 1u : 0u;
  s_item = 0u;
  __syncthreads();
  for (uint32_t j = 0; j < kXcds; ++j) {
    const uint32_t k = (home + j) % kXcds;
    const uint32_t first = k * q + min(k, r), len = q + (k < r ? 1u : 0u);
    for (;;) {
      const uint32_t c = atomicAdd(map.queue + k * kQueueStride, one);
      atomicAdd(&s_item, one * c);
      __syncthreads();
      const uint32_t i = __builtin_amdgcn_readfirstlane(s_item);
      __syncthreads();  // every wave holds the item before the word is cleared
      s_item = 0u;
      __syncthreads();  // ... and cleared before the next claim adds to it
      if (i >= len) break;
      tv_batch_item<H, SEQ, FINAL, TV2, FGP, BF, SP>(args, map, first + i);
    }
  }
  // every block passes here once, after its last claim on every counter
  if (threadIdx.x == 0 && atomicAdd(map.queue + kXcds * kQueueStride, 1u) == gridDim.x - 1)
    for (uint32_t k = 0; k <= kXcds; ++k) atomicExch(map.queue + k * kQueueStride, 0u);
}

template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
static void launch_batched(dim3 g, const TvPassArgs* a, const BatchMap& map, hipStream_t s) {
  const dim3 b(kTvWaves * 64);
  if (map.queue != nullptr)
    hipLaunchKernelGGL((k_tv_pass_q<H, SEQ, FINAL, TV2, FGP, BF, SP>), dim3(std::max(1, std::min<int>(g.x, map.grid))), b,
                       0, s, a, map);
  else hipLaunchKernelGGL((k_tv_pass_b<H, SEQ, FINAL, TV2, FGP, BF, SP>), g, b, 0, s, a, map);
}

// Kernel selection for one fusion depth: form, final / dual pass, 2D or 3D TV, FGP
// (dual passes of depth-2 tiles only), bfloat16 dual, row-compressed output
// (final passes with an FP32 dual only), single or batched form.  One source
// file per depth instantiates it.
struct TvSelect {
  bool batch, final_pass, tv2, fgp, bf16, sparse, low, seq;   // low: tiles of kTvSmallQ rows a lane
};
template <int H, bool SEQ, bool FINAL, bool TV2, bool FGP, bool BF, bool SP>
static void launch_tv_kernel(bool batch, dim3 g, const TvPassArgs* a, const BatchMap& map, hipStream_t s) {
  if (batch) launch_batched<H, SEQ, FINAL, TV2, FGP, BF, SP>(g, a, map, s);
  else hipLaunchKernelGGL((k_tv_pass<H, SEQ, FINAL, TV2, FGP, BF, SP>), g, dim3(kTvWaves * 64), 0, s, *a);
}
// Forms that exist: a step of FGP never fills the pipeline, and the final pass of depth 4
// takes SEQ only for few planes, in a launch of its own on dense iterates (a row store
// would spill).
__host__ __device__ constexpr bool tv_has_seq(int H, bool final_pass, bool single_dense) {
  return H < kTvLevelsMax || !final_pass || single_dense;
}

template <int H, bool SEQ, bool TV2>
static void launch_tv_dim(const TvSelect& k, dim3 g, const TvPassArgs* a, const BatchMap& map, hipStream_t s) {
  if constexpr (H == kTvDefaultLevels) {
    if (k.low) {   // (single launches with an FP32 dual only)
      const dim3 b(kTvWaves * 64);
      if (k.final_pass) hipLaunchKernelGGL((k_tv_pass<H, SEQ, true, TV2, false, false, false, kTvSmallQ>), g, b, 0, s, *a);
      else hipLaunchKernelGGL((k_tv_pass<H, SEQ, false, TV2, false, false, false, kTvSmallQ>), g, b, 0, s, *a);
      return;
    }
  }
  if (k.final_pass) {
    if constexpr (SEQ && H == kTvLevelsMax) {
      const dim3 b(kTvWaves * 64);
      if (k.bf16) hipLaunchKernelGGL((k_tv_pass<H, SEQ, true, TV2, false, true, false>), g, b, 0, s, *a);
      else hipLaunchKernelGGL((k_tv_pass<H, SEQ, true, TV2, false, false, false>), g, b, 0, s, *a);
    } else {
      if (k.sparse && !k.bf16) launch_tv_kernel<H, SEQ, true, TV2, false, false, true>(k.batch, g, a, map, s);
      else if (k.bf16) launch_tv_kernel<H, SEQ, true, TV2, false, true, false>(k.batch, g, a, map, s);
      else launch_tv_kernel<H, SEQ, true, TV2, false, false, false>(k.batch, g, a, map, s);
    }
    return;
  }
  if constexpr (H == 2 && SEQ) {
    if (k.fgp) {
      if (k.bf16) launch_tv_kernel<H, SEQ, false, TV2, true, true, false>(k.batch, g, a, map, s);
      else launch_tv_kernel<H, SEQ, false, TV2, true, false, false>(k.batch, g, a, map, s);
      return;
    }
  }
  if (k.bf16) launch_tv_kernel<H, SEQ, false, TV2, false, true, false>(k.batch, g, a, map, s);
  else launch_tv_kernel<H, SEQ, false, TV2, false, false, false>(k.batch, g, a, map, s);
}
template <int H>
void launch_tv_depth(const TvSelect& k, dim3 g, const TvPassArgs* a, const BatchMap& map, hipStream_t s) {
  if (k.seq) {
    if (k.tv2) launch_tv_dim<H, true, true>(k, g, a, map, s);
    else launch_tv_dim<H, true, false>(k, g, a, map, s);
  } else {
    if (k.tv2) launch_tv_dim<H, false, true>(k, g, a, map, s);
    else launch_tv_dim<H, false, false>(k, g, a, map, s);
  }
}

}  // namespace rihvr
