// Gradient-projection TV prox and objective partials, templated on the
// element type T (float, double) and the number of parts NP (1: real object,
// 2: complex object).  They serve the complex object in FP32 and every FP64
// plan.
//
// Complex object.  A complex plan holds the object as two real volumes of nz
// planes, the real parts and then the imaginary parts ([2][nz][ny][nx]).  The
// hologram model and its adjoint need no kernels of their own:
// Re(IFFT2(FFT2(i y) H_j)) is the real model with H_j multiplied by i, a
// carrier phase advanced by a quarter cycle, so the plan gives its second nz
// planes the carriers c_j + 1/4 and the real kernels run on all 2 nz planes
// (their adjoint then returns the real and imaginary parts of A^T r).  What is
// complex is the regulariser (section "Methodology"): the l1 norm of Eq. (3)
// sums moduli, the TV of Eq. (4) takes the modulus of complex differences, and
// the soft threshold of Eq. (8) shrinks the modulus and keeps the phase.
//
// The TV prox is gradient projection on the dual, one value per part and
// direction, projected jointly on the unit ball.  One launch takes up to two
// (FP64) or three (FP32) steps, streamed along z, and writes the other of two
// dual sets, so the sets alternate launch by launch.
// The last launch forms u once more and writes the threshold (real: max(u -
// thr, 0) or the signed form; complex: the shrinkage of the modulus), with the
// occupancy flags.
#include <hip/hip_runtime.h>

#include <utility>

#include "rihvr_internal.h"

namespace rihvr {
namespace {

constexpr int kGThreads = 256;

template <class T>
struct GpArgs {
  const T* v;            // input [NP][nz][ny][nx]; nullptr: vol[st->prev]
  T* x;                  // output; nullptr: vol[st->next]
  T* vol[3];
  const SolveState* st;
  T* p[3];               // dual read by a step and by the final launch, [NP][nz][ny][nx] each
                         // (p[2] unused in 2D)
  T* q[3];               // dual written by a step (the two sets alternate)
  uint8_t* rowflag;      // nullable: [NP nz][ny], set where a row of a part is non-zero
  uint8_t* planeflag;    // [NP nz]
  int nx, ny, nz;        // nz: planes of one part
  int tv2;
  int nonneg;            // real object: x >= 0
  int first;             // the dual is zero (no step taken yet)
  int levels;            // steps of this launch
  int gx, gy, zchunk;    // tiles along x and y, planes per block
  T tau, c, thr;
};

__device__ __forceinline__ bool done(const SolveState* st) { return st != nullptr && st->done != 0; }

template <class T>
__device__ __forceinline__ const T* in_of(const GpArgs<T>& a) {
  return a.v != nullptr ? a.v : pick3<T>(a.vol[0], a.vol[1], a.vol[2], a.st->prev);
}
template <class T>
__device__ __forceinline__ T* out_of(const GpArgs<T>& a) {
  return a.x != nullptr ? a.x : pick3<T>(a.vol[0], a.vol[1], a.vol[2], a.st->next);
}

__device__ __forceinline__ float fmaT(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float sqrtT(float a) { return sqrtf(a); }
__device__ __forceinline__ double sqrtT(double a) { return sqrt(a); }

// -(D^T p) at voxel i of the part starting at offset o: the backward
// differences of the dual, zero where the forward difference is not defined.
template <class T>
__device__ __forceinline__ T neg_div(const GpArgs<T>& a, size_t i, size_t o, int x, int y, int z) {
  const size_t plane = (size_t)a.nx * a.ny;
  const T* px = a.p[0] + o;
  const T* py = a.p[1] + o;
  T d = (x + 1 < a.nx ? px[i] : T(0)) - (x > 0 ? px[i - 1] : T(0));
  d += (y + 1 < a.ny ? py[i] : T(0)) - (y > 0 ? py[i - a.nx] : T(0));
  if (!a.tv2) {
    const T* pz = a.p[2] + o;
    d += (z + 1 < a.nz ? pz[i] : T(0)) - (z > 0 ? pz[i - plane] : T(0));
  }
  return d;
}

// Up to LV gradient-projection steps in one launch, streamed along z.  A
// wavefront holds 64 points along x (a lane each) of Q rows, NW wavefronts a
// 64 x 16 tile; step l works one plane behind step l - 1 and keeps, per point,
// its previous plane's dual and u in registers.  Neighbours along x come by DPP
// wave shifts, along y from the lane's other row or through LDS rows, one
// barrier per step and plane.  Points within LV of the tile's edge are computed
// but not stored, and a chunk of planes has LV planes of margin; a chunk's
// planes are read through buffer descriptors (0 outside the volume), one plane
// ahead.  State below the volume starts at zero and the dual's component along
// an axis is exactly zero on that axis' last plane, so z needs no masks; x / y
// masks are compiled only into tiles at the volume's edge (EDGE), the z component into
// the 3D form (TV3).
//
// Bound by the latency of its loads and of the exchange at each barrier, at
// large sizes by memory: v and the dual in and out once per LV steps, 56 B per
// complex FP32 voxel, the reads 16 / (16 - 2 LV) times over for the halo.  Two
// blocks of eight wavefronts a compute unit hide that best: 512 x 384 x 48
// complex, 20 steps, 1588 us with LV = 3, 1743 with 2 (1024^2 x 64: 9.2 and 14.7
// ms); one block of sixteen wavefronts and 32 rows 1613 (9.1 ms), LV = 4 spills
// (2626).  FP64 has registers for LV = 2.  Against a pair of steps through LDS
// with six stages and five barriers a plane (FP64: a step): 2934 us; FP64 real
// 192 x 128 x 24, 10 steps, 450 -> 123 us; 256^2 x 48 complex FP64, 10 steps, 1559 ->
// 563, in 2D 1092 -> 333.  A single step takes tiles with a halo of one, and no dual is
// loaded where it is zero: one step at 512^2 x 32 in 2D, complex FP64, 333 -> 193 us.
constexpr unsigned kGpOff = 0x40000000u;   // past every plane, also when two are added

__device__ __forceinline__ int dpp_left(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_right(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_same(int v) { return __builtin_amdgcn_mov_dpp(v, 0xE4, 0xf, 0xf, false); }
#define RIHVR_LANES(name, op)                                                            \
  __device__ __forceinline__ float name(float v) { return __int_as_float(op(__float_as_int(v))); } \
  __device__ __forceinline__ double name(double v) {                                     \
    return __hiloint2double(op(__double2hiint(v)), op(__double2loint(v)));               \
  }
RIHVR_LANES(from_left, dpp_left)     // lane i <- lane i - 1 (0 at lane 0)
RIHVR_LANES(from_right, dpp_right)   // lane i <- lane i + 1 (0 at lane 63)
RIHVR_LANES(kept_copy, dpp_same)     // a copy that the compiler keeps: the loaded registers are free for the next plane
#undef RIHVR_LANES

template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gp_rsrc(const T* base, size_t plane, size_t sz, bool on) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base) + plane * sz, (short)0, on ? (int)(sz * sizeof(T)) : 0,
                                           0x00020000);
}
typedef unsigned int gp_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void gp_ld(float& v, __amdgpu_buffer_rsrc_t r, unsigned off) {
  v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ void gp_ld(double& v, __amdgpu_buffer_rsrc_t r, unsigned off) {
  const gp_u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
  v = __hiloint2double((int)u.y, (int)u.x);
}
__device__ __forceinline__ void gp_st(float v, __amdgpu_buffer_rsrc_t r, unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)off, 0, 0);
}
__device__ __forceinline__ void gp_st(double v, __amdgpu_buffer_rsrc_t r, unsigned off) {
  const gp_u32x2 u = {(unsigned)__double2loint(v), (unsigned)__double2hiint(v)};
  __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)off, 0, 0);
}

// 1 / max(1, sqrt(n2)).  FP32: the hardware's reciprocal square root (1 ulp)
// with one Newton step (not where n2 is infinite: 0, as 1 / sqrt(n2)).
__device__ __forceinline__ float proj_scale(float n2) {
  const float r = __builtin_amdgcn_rsqf(n2);
  const float e = fmaf(-n2 * r, r, 1.f);
  const float q = fmaf(0.5f * r, e, r);
  return n2 > 1.f ? (n2 < __builtin_huge_valf() ? q : r) : 1.f;
}
// FP64: the hardware's estimate (24 bits) with one step of third order, within
// 2 ulp, for a square root and a division (prox of 192 x 128 x 24, 10 steps, 153 ->
// 131 us; the solves' distance from the oracle does not change).
__device__ __forceinline__ double proj_scale(double n2) {
  const double r = __builtin_amdgcn_rsq(n2);
  const double e = fma(-n2 * r, r, 1.0);
  const double q = fma(r * e, fma(0.375, e, 0.5), r);
  return n2 > 1.0 ? (n2 < __builtin_huge_val() ? q : r) : 1.0;
}

// Rows of a lane and wavefronts of a tile (FP64 complex: a row per lane), steps per launch.
template <class T, int NP>
constexpr int gp_q() { return sizeof(T) * NP > 8 ? 1 : 2; }
template <class T, int NP>
constexpr int gp_waves() { return sizeof(T) * NP > 8 ? 16 : 8; }
template <class T, int NP>
constexpr int gp_rows() { return gp_q<T, NP>() * gp_waves<T, NP>(); }
template <class T>
constexpr int gp_levels() { return sizeof(T) == 4 ? 3 : 2; }

template <class T, int NP, int LV, bool TV3, bool EDGE>
__device__ __forceinline__ void gp_pass_body(const GpArgs<T>& a, int bx, int by, int zb, int ze,
                                             T (*s_py)[2][NP][gp_waves<T, NP>()][64],
                                             T (*s_ut)[2][NP][gp_waves<T, NP>()][64]) {
  constexpr int NW = gp_waves<T, NP>(), Q = gp_q<T, NP>(), RY = gp_rows<T, NP>(), H = LV, ND = TV3 ? 3 : 2;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const size_t sz = (size_t)nx * ny;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool pre = !a.first;
  const int L = a.levels;
  const T tau = a.tau, cc = a.c;
  const T* v = in_of(a);
  const int x = bx * (64 - 2 * H) - H + lane;
  const bool inx = !EDGE || (x >= 0 && x < nx);
  const bool xlo = !EDGE || x > 0, xhi = !EDGE || x + 1 < nx;
  bool ylo[Q], yhi[Q];
  unsigned offl[Q], offs[Q];   // in-plane byte offsets of loads and stores (kGpOff and above: none)
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int r = wv * Q + q, y = by * (RY - 2 * H) - H + r;
    const bool iny = !EDGE || (y >= 0 && y < ny);
    ylo[q] = !EDGE || y > 0;
    yhi[q] = !EDGE || y + 1 < ny;
    offl[q] = inx && iny ? (unsigned)(y * nx + x) * (unsigned)sizeof(T) : kGpOff;
    offs[q] = inx && iny && lane >= H && lane < 64 - H && r >= H && r < RY - H ? offl[q] : kGpOff;
  }
  const int M = TV3 ? L : 0;
  const int zs = max(0, zb - M), zl = min(nz, ze + M);

  struct Plane {
    T v[Q][NP], p[Q][ND][NP];
  };
  auto load_plane = [&](Plane& r, int z) __attribute__((always_inline)) {
#pragma unroll
    for (int part = 0; part < NP; ++part) {
      const __amdgpu_buffer_rsrc_t rv = gp_rsrc(v, (size_t)part * nz + z, sz, true);
#pragma unroll
      for (int q = 0; q < Q; ++q) gp_ld(r.v[q][part], rv, offl[q]);
    }
    if (!pre) return;   // (r.p stays zero)
#pragma unroll
    for (int part = 0; part < NP; ++part) {
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const __amdgpu_buffer_rsrc_t rp = gp_rsrc<T>(a.p[d], (size_t)part * nz + z, sz, true);
#pragma unroll
        for (int q = 0; q < Q; ++q) gp_ld(r.p[q][d][part], rp, offl[q]);
      }
    }
  };
  // per step: the previous plane's dual and u; v of the planes that steps 1.. are at
  T Pp[LV][Q][ND][NP], Up[LV][Q][NP], V[LV][Q][NP];
#pragma unroll
  for (int l = 0; l < LV; ++l)
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int part = 0; part < NP; ++part) {
#pragma unroll
        for (int d = 0; d < ND; ++d) Pp[l][q][d][part] = T(0);
        Up[l][q][part] = V[l][q][part] = T(0);
      }
  T C[Q][ND][NP];
  Plane P;
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int part = 0; part < NP; ++part) C[q][d][part] = P.p[q][d][part] = T(0);
  // dual step at the plane held in Pp / Up, whose next plane's u is un (hz: it exists), into o
  auto step = [&](int l, int par, bool hz, const T (&un)[Q][NP], T (&o)[Q][ND][NP]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      T w[ND][NP];
      T n2 = T(0);
#pragma unroll
      for (int part = 0; part < NP; ++part) {
        const T u0 = Up[l][q][part];
        const T ux = from_right(u0);
        const T uy = q < Q - 1 ? Up[l][q < Q - 1 ? q + 1 : q][part] : s_ut[l][par ^ 1][part][wv < NW - 1 ? wv + 1 : wv][lane];
        const T g[3] = {xhi ? ux - u0 : T(0), yhi[q] ? uy - u0 : T(0), hz ? un[q][part] - u0 : T(0)};
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          w[d][part] = fmaT(cc, g[d], Pp[l][q][d][part]);
          n2 = fmaT(w[d][part], w[d][part], n2);
        }
      }
      const T sc = proj_scale(n2);
#pragma unroll
      for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int part = 0; part < NP; ++part) o[q][d][part] = w[d][part] * sc;
    }
  };
  load_plane(P, zs);
  const int nsteps = zl - zs + L;   // the last output leaves at s = nsteps - 1
  for (int s = 0; s < nsteps; ++s) {
    const int par = s & 1, a1 = zs + s;
    if (a1 < zl) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int part = 0; part < NP; ++part) {
          V[0][q][part] = kept_copy(P.v[q][part]);
#pragma unroll
          for (int d = 0; d < ND; ++d) C[q][d][part] = kept_copy(P.p[q][d][part]);
        }
      if (a1 + 1 < zl) load_plane(P, a1 + 1);
    }
#pragma unroll
    for (int l = 0; l < LV; ++l) {
      const int z = a1 - l;   // plane of step l
      if (l >= L) continue;
      const bool arrives = z >= zs && z < zl;
#pragma unroll
      for (int part = 0; part < NP; ++part) s_py[l][par][part][wv][lane] = C[Q - 1][1][part];
      __syncthreads();
      if (arrives) {
        T un[Q][NP];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int part = 0; part < NP; ++part) {
            const T cx = C[q][0][part], cy = C[q][1][part];
            const T pxm = from_left(cx);
            const T pym = q > 0 ? C[q > 0 ? q - 1 : 0][1][part] : s_py[l][par][part][wv > 0 ? wv - 1 : 0][lane];
            T d = (xhi ? cx : T(0)) - (xlo ? pxm : T(0));
            d += (yhi[q] ? cy : T(0)) - (ylo[q] ? pym : T(0));
            if constexpr (TV3) d += C[q][2][part] - Pp[l][q][2][part];
            un[q][part] = fmaT(tau, d, V[l][q][part]);
          }
        T O[Q][ND][NP];
        step(l, par, true, un, O);
#pragma unroll
        for (int part = 0; part < NP; ++part) s_ut[l][par][part][wv][lane] = un[0][part];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int part = 0; part < NP; ++part) {
            Up[l][q][part] = un[q][part];
#pragma unroll
            for (int d = 0; d < ND; ++d) {
              Pp[l][q][d][part] = C[q][d][part];
              C[q][d][part] = O[q][d][part];   // (of no plane when z == zs: not used)
            }
          }
      } else if (z == zl) {   // the last plane: no plane above it
        step(l, par, false, Up[l], C);
      }
    }
    const int m = a1 - L;
    const bool on = m >= zb && m < ze;
#pragma unroll
    for (int part = 0; part < NP; ++part)
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const __amdgpu_buffer_rsrc_t ro = gp_rsrc<T>(a.q[d], (size_t)part * nz + (on ? m : 0), sz, on);
#pragma unroll
        for (int q = 0; q < Q; ++q) gp_st(C[q][d][part], ro, offs[q]);
      }
#pragma unroll
    for (int l = LV - 1; l > 0; --l)
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int part = 0; part < NP; ++part) V[l][q][part] = V[l - 1][q][part];
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <class T, int NP, int LV, bool TV3>
__global__ void __launch_bounds__((gp_waves<T, NP>() * 64), 4) k_gp_pass(GpArgs<T> a) {
  constexpr int NW = gp_waves<T, NP>(), RY = gp_rows<T, NP>();
  __shared__ T s_py[LV][2][NP][NW][64];   // bottom-row p_y of every wavefront, by step and parity
  __shared__ T s_ut[LV][2][NP][NW][64];   // top-row u
  if (done(a.st)) return;
  // Where a plane's tiles alone occupy the units, neighbouring ones meet in one
  // XCD's L2 (prox, 20 steps: 1024^2 x 256 complex 48.8 -> 41.5 ms, 512 x 384 x 48
  // 1587 -> 1514 us, 1024^2 x 64 9.19 -> 9.39 ms); smaller planes, cut into many
  // chunks, take the hardware's order (128^2 x 16: 104 us, 123 the other way).
  const int t = (int)(a.gx * a.gy >= 256 ? xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x);
  const int tile = t % (a.gx * a.gy), zb = t / (a.gx * a.gy) * a.zchunk;
  const int bx = tile % a.gx, by = tile / a.gx;
  const int x0 = bx * (64 - 2 * LV) - LV, y0 = by * (RY - 2 * LV) - LV;
  const bool interior = x0 >= 1 && x0 + 64 <= a.nx - 1 && y0 >= 1 && y0 + RY <= a.ny - 1;
  const int ze = min(a.nz, zb + a.zchunk);
  if (interior) gp_pass_body<T, NP, LV, TV3, false>(a, bx, by, zb, ze, s_py, s_ut);
  else gp_pass_body<T, NP, LV, TV3, true>(a, bx, by, zb, ze, s_py, s_ut);
}

// u once more, then the threshold and the flags.  In place is allowed (a
// voxel reads only its own v).
template <class T, int NP>
__global__ void __launch_bounds__(kGThreads) k_gp_final(GpArgs<T> a) {
  if (done(a.st)) return;
  const size_t n = (size_t)a.nx * a.ny * a.nz;
  const T* v = in_of(a);
  T* xo = out_of(a);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(i % a.nx), y = (int)((i / a.nx) % a.ny), z = (int)(i / ((size_t)a.nx * a.ny));
    T u[NP], r[NP];
    T m2 = T(0);
#pragma unroll
    for (int part = 0; part < NP; ++part) {
      u[part] = v[part * n + i];
      if (!a.first) u[part] = fmaT(a.tau, neg_div(a, i, part * n, x, y, z), u[part]);
      m2 = fmaT(u[part], u[part], m2);
    }
    if constexpr (NP == 1) {
      if (a.nonneg) {
        r[0] = u[0] - a.thr > T(0) ? u[0] - a.thr : T(0);
      } else {
        const T m = u[0] < T(0) ? -u[0] : u[0];
        r[0] = m > a.thr ? (u[0] < T(0) ? -(m - a.thr) : m - a.thr) : T(0);
      }
    } else {
      const T mod = sqrtT(m2);
      const T s = mod > a.thr ? T(1) - a.thr / mod : T(0);
#pragma unroll
      for (int part = 0; part < NP; ++part) r[part] = s * u[part];
    }
#pragma unroll
    for (int part = 0; part < NP; ++part) {
      xo[part * n + i] = r[part];
      if (a.rowflag != nullptr && r[part] != T(0)) {
        a.rowflag[(size_t)(part * a.nz + z) * a.ny + y] = 1;
        a.planeflag[part * a.nz + z] = 1;
      }
    }
  }
}

// Per-block FP64 partials of sum |x| and TV(x) (the solver's iterate x_it
// before the scalar kernel of its iteration, or x0 outside one).
template <class T>
struct ObjPartArgs {
  const T* x0; const T* x1; const T* x2;
  const SolveState* st;
  double* psum; double* ptv;
  int nx, ny, nz;        // nz: planes of one part
  int tv2;
};

template <class T, int NP>
__global__ void __launch_bounds__(kGThreads) k_gp_obj(ObjPartArgs<T> a) {
  if (done(a.st)) return;
  __shared__ double red[2][kGThreads / 64];
  const T* __restrict__ xv = a.st != nullptr ? pick3<const T>(a.x0, a.x1, a.x2, a.st->it % 3) : a.x0;
  const size_t n = (size_t)a.nx * a.ny * a.nz;
  const size_t plane = (size_t)a.nx * a.ny;
  double s_acc = 0.0, t_acc = 0.0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(i % a.nx), y = (int)((i / a.nx) % a.ny), z = (int)(i / plane);
    T g2 = T(0), m2 = T(0);
#pragma unroll
    for (int part = 0; part < NP; ++part) {
      const T* u = xv + part * n;
      const T c = u[i];
      m2 = fmaT(c, c, m2);
      const T gx = x + 1 < a.nx ? u[i + 1] - c : T(0);
      const T gy = y + 1 < a.ny ? u[i + a.nx] - c : T(0);
      const T gz = (!a.tv2 && z + 1 < a.nz) ? u[i + plane] - c : T(0);
      g2 = fmaT(gx, gx, fmaT(gy, gy, fmaT(gz, gz, g2)));
    }
    s_acc += (double)sqrtT(m2);
    t_acc += (double)sqrtT(g2);
  }
  for (int off = 32; off > 0; off >>= 1) {
    s_acc += __shfl_down(s_acc, off, 64);
    t_acc += __shfl_down(t_acc, off, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wv] = s_acc;
    red[1][wv] = t_acc;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0, t = 0.0;
    for (int w = 0; w < kGThreads / 64; ++w) {
      s += red[0][w];
      t += red[1][w];
    }
    a.psum[blockIdx.x] = s;
    a.ptv[blockIdx.x] = t;
  }
}

int ggrid(size_t n) {
  const size_t b = (n + kGThreads - 1) / kGThreads;
  return (int)(b > 8192 ? 8192 : (b == 0 ? 1 : b));
}

// Planes per block of a pass: the cut whose rounds (16 wavefronts a compute unit: two
// blocks of eight, one of sixteen) times a block's march, its planes and `extra` of
// margin and pipeline (3 LV, in 2D without margin LV), is shortest.  FP64 in 2D, 10 steps,
// without the LV: 1024^2 x 8 real 544 us, now 400; complex 1509 and 958.
int gp_zchunk(int tiles, int nz, int extra, int slots) {
  int best = nz;
  long best_t = -1;
  for (int nc = 1; nc <= nz; ++nc) {
    const int zc = (nz + nc - 1) / nc;
    const long blocks = (long)tiles * ((nz + zc - 1) / zc);
    const long t = (blocks + slots - 1) / slots * (zc + extra);
    if (best_t < 0 || t < best_t) {
      best_t = t;
      best = zc;
    }
  }
  return best;
}

// A launch of up to LV steps.
template <class T, int NP, int LV>
void launch_gp(GpArgs<T> a, int cus, hipStream_t s) {
  constexpr int RY = gp_rows<T, NP>(), NW = gp_waves<T, NP>();
  a.gx = (a.nx + 64 - 2 * LV - 1) / (64 - 2 * LV);
  a.gy = (a.ny + RY - 2 * LV - 1) / (RY - 2 * LV);
  a.zchunk = gp_zchunk(a.gx * a.gy, a.nz, a.tv2 ? LV : 3 * LV, (cus > 0 ? cus : 256) * (16 / NW));
  const dim3 g(a.gx * a.gy * ((a.nz + a.zchunk - 1) / a.zchunk)), b(NW * 64);
  if (a.tv2) hipLaunchKernelGGL((k_gp_pass<T, NP, LV, false>), g, b, 0, s, a);
  else hipLaunchKernelGGL((k_gp_pass<T, NP, LV, true>), g, b, 0, s, a);
}

// K steps, LV a launch (a single step left over on tiles with a halo of one),
// alternating between the dual sets a.p and a.q, then the final launch on the set the
// last one wrote.
template <class T, int NP>
hipError_t run_gp(GpArgs<T> a, int K, int cus, hipStream_t s, int* launches) {
  constexpr int LV = gp_levels<T>();
  const dim3 g(ggrid((size_t)a.nx * a.ny * a.nz)), b(kGThreads);
  int nl = 0;
  for (int k = 0; k < K;) {
    a.first = k == 0 ? 1 : 0;
    a.levels = K - k < LV ? K - k : LV;
    if (a.levels == 1) launch_gp<T, NP, 1>(a, cus, s);
    else launch_gp<T, NP, LV>(a, cus, s);
    k += a.levels;
    for (int d = 0; d < 3; ++d) std::swap(a.p[d], a.q[d]);
    ++nl;
  }
  a.first = K == 0 ? 1 : 0;
  hipLaunchKernelGGL((k_gp_final<T, NP>), g, b, 0, s, a);
  if (launches) *launches = nl + 1;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_cprox(const ProxArgs& pa, hipStream_t s, int* launches) {
  GpArgs<float> a{};
  a.v = pa.v;
  a.x = pa.x;
  for (int k = 0; k < 3; ++k) a.vol[k] = pa.vol[k];
  a.st = pa.st;
  for (int k = 0; k < 3; ++k) {
    a.p[k] = pa.pa[k];
    a.q[k] = pa.pb[k];
  }
  a.rowflag = pa.rowflag;
  a.planeflag = pa.planeflag;
  a.nx = pa.nx;
  a.ny = pa.ny;
  a.nz = pa.nz / 2;
  a.tv2 = pa.tv2 ? 1 : 0;
  const double tau = pa.step * pa.tv;
  const int K = (tau > 0.0 && pa.inner_iters > 0) ? pa.inner_iters : 0;
  a.tau = (float)tau;
  a.c = K > 0 ? (float)(1.0 / ((a.tv2 ? 8.0 : 12.0) * tau)) : 0.f;
  a.thr = (float)(pa.step * pa.l1);
  return run_gp<float, 2>(a, K, pa.cus, s, launches);
}

hipError_t launch_cobj(const ObjArgs& oa, int nblocks, hipStream_t s) {
  ObjPartArgs<float> a{};
  a.x0 = oa.x0;
  a.x1 = oa.x1;
  a.x2 = oa.x2;
  a.st = oa.st;
  a.psum = oa.psum;
  a.ptv = oa.ptv;
  a.nx = oa.nx;
  a.ny = oa.ny;
  a.nz = oa.nz / 2;
  a.tv2 = oa.tv2;
  hipLaunchKernelGGL((k_gp_obj<float, 2>), dim3(nblocks > 0 ? nblocks : 1), dim3(kGThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_prox64(const Prox64Args& pa, hipStream_t s) {
  GpArgs<double> a{};
  a.v = pa.v;
  a.x = pa.x;
  for (int k = 0; k < 3; ++k) {
    a.p[k] = pa.p[k];
    a.q[k] = pa.p2[k];
  }
  a.nx = pa.nx;
  a.ny = pa.ny;
  a.nz = pa.nz;
  a.tv2 = pa.tv2;
  a.nonneg = pa.nonneg;
  const double tau = pa.step * pa.tv;
  const int K = (tau > 0.0 && pa.inner_iters > 0) ? pa.inner_iters : 0;
  a.tau = tau;
  a.c = K > 0 ? 1.0 / ((pa.tv2 ? 8.0 : 12.0) * tau) : 0.0;
  a.thr = pa.step * pa.l1;
  return pa.parts == 2 ? run_gp<double, 2>(a, K, pa.cus, s, nullptr) : run_gp<double, 1>(a, K, pa.cus, s, nullptr);
}

hipError_t launch_obj64(const double* x, int nx, int ny, int nz, int parts, int tv2, double* psum, double* ptv,
                        int nblocks, hipStream_t s) {
  ObjPartArgs<double> a{};
  a.x0 = a.x1 = a.x2 = x;
  a.psum = psum;
  a.ptv = ptv;
  a.nx = nx;
  a.ny = ny;
  a.nz = nz;
  a.tv2 = tv2;
  if (parts == 2) hipLaunchKernelGGL((k_gp_obj<double, 2>), dim3(nblocks), dim3(kGThreads), 0, s, a);
  else hipLaunchKernelGGL((k_gp_obj<double, 1>), dim3(nblocks), dim3(kGThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace rihvr
