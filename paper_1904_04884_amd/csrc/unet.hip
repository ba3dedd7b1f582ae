// Warm-start 3D U-Net kernels for gfx950: BF16 activations and weights, FP32
// accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Activations are channels-last, [z][y][x][c]; the two halves of a
// concatenation are buffers of their own.  Every convolution-like layer is a
// matrix product: row r is an output voxel, the reduction index k = t*C + c runs
// over taps t and input channels c.  The 3x3x3 layers read their operand from a
// haloed box in LDS (k_conv3); the others gather it from a source voxel chosen by
// the layer's mode (k_gather_gemm).  Weights are packed as B[t][n][c] (n the
// output channel, c contiguous) so each lane loads 8 consecutive reduction values
// with one 16-byte load.
//
// MFMA 16x16x32 operand layout (per wavefront of 64 lanes, lane l):
//   A (16 x 32): row l % 16, reduction elements 8 (l / 16) .. 8 (l / 16) + 7
//   B (32 x 16): column l % 16, reduction elements 8 (l / 16) .. + 7
//   D (16 x 16): rows 4 (l / 16) .. 4 (l / 16) + 3, column l % 16
#include <algorithm>
#include <type_traits>

#include "rihvr_internal.h"
#include "unet_internal.h"

namespace rihvr {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even (finite inputs)
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Two values rounded and packed (the first in the low half).
__device__ __forceinline__ uint32_t bf_pack(float a, float b) {
  uint32_t u = __float_as_uint(a), v = __float_as_uint(b);
  u += 0x7fffu + ((u >> 16) & 1u);
  v += 0x7fffu + ((v >> 16) & 1u);
  return __builtin_amdgcn_perm(v, u, 0x07060302u);
}
// Four packed values, zero where the mask's is not > 0.
__device__ __forceinline__ u32x2 bf_mask(u32x2 o, u32x2 m) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint32_t lo = bf2f((uint16_t)m[k]) > 0.f ? 0xffffu : 0u, hi = bf2f((uint16_t)(m[k] >> 16)) > 0.f ? 0xffff0000u : 0u;
    o[k] &= lo | hi;
  }
  return o;
}

// Planes as buffer resources: a read past the given bytes returns 0, a store
// there is dropped (kBufOff lies past every plane).
constexpr uint32_t kBufOff = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Row coordinates of one lane, computed once: the source voxel of a tap is
// then found with adds and compares only (no 64-bit division per k-step).
struct GgRow {
  int x, y, z;
  bool ok;
};
__device__ __forceinline__ GgRow gg_row(const GatherGemmArgs& a, long r, long nrows) {
  GgRow g;
  g.ok = r < nrows;
  const uint32_t rr = g.ok ? (uint32_t)r : 0u;   // fewer than 2^31 rows (launch_gather_gemm)
  const uint32_t zy = rr / (uint32_t)a.W;
  g.x = (int)(rr - zy * a.W);
  g.z = (int)(zy / (uint32_t)a.H);
  g.y = (int)(zy - g.z * (uint32_t)a.H);
  return g;
}

// Source voxel (linear index at the source resolution) of a row for tap t, or -1.
template <int MODE>
__device__ __forceinline__ long gg_source_m(const GatherGemmArgs& a, const GgRow& g, int t) {
  const int H = a.H, W = a.W;  // row grid
  if constexpr (MODE == GG_UP_BWD) {
    // row (z, y, x) is a coarse voxel; tap t = dz*4 + dy*2 + dx selects the fine voxel
    const int zz = 2 * g.z + (t >> 2), yy = 2 * g.y + ((t >> 1) & 1), xx = 2 * g.x + (t & 1);
    return ((long)zz * (2 * H) + yy) * (2 * W) + xx;
  } else {  // GG_POINT
    return ((long)g.z * H + g.y) * W + g.x;
  }
}
// Load target of switched-off lanes (zero-initialised device memory): operand
// loads are selects of an address, never branches, so that the loads of the
// next reduction step stay in flight under the MFMAs of this one.
__device__ uint4 g_gg_zero;

// Block: 4 wavefronts x (16 RT) rows; every wavefront computes all NB column
// tiles of its RT row tiles, so a B fragment (weights) feeds RT MFMAs and an A
// fragment (gathered activations) feeds NB.  The reduction index k = t C + c
// advances by 32 per step with t, c updated incrementally.  The operands of
// step k + 32 are loaded while the MFMAs of step k run (two register sets used
// in turn; B is prefetched too while it is small).
template <int NB, int RT, int MODE>
__global__ void __launch_bounds__(256) k_gather_gemm(GatherGemmArgs a) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const long row0 = ((long)blockIdx.x * 4 + wv) * (16 * RT);
  const long nrows = (long)a.D * a.H * a.W;
  const int kq = (lane >> 4) * 8;       // reduction offset of this lane within a 32-chunk
  const int K = a.T * a.C;
  GgRow rows[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) rows[i] = gg_row(a, row0 + i * 16 + (lane & 15), nrows);
  f32x4 acc[RT][NB];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* __restrict__ src = a.src;
  const uint16_t* __restrict__ wt = a.wt;
  const uint4* zero = &g_gg_zero;
  constexpr bool PB = NB <= 4;   // B prefetched with A
  constexpr int NBP = PB ? NB : 1;
  struct Step {                  // operand position of one reduction step
    int t, c;
    bool kin;
  };
  auto next = [&](Step st) {
    st.c += 32;
    while (st.c >= a.C) {
      st.c -= a.C;
      ++st.t;
    }
    st.kin = st.t * a.C + st.c < K;
    return st;
  };
  auto ld_a = [&](int i, const Step& st) -> uint4 {
    const long sv = gg_source_m<MODE>(a, rows[i], st.t);
    const bool on = st.kin && rows[i].ok && sv >= 0;
    return *(on ? reinterpret_cast<const uint4*>(src + sv * a.src_cs + st.c) : zero);
  };
  auto ld_b = [&](int j, const Step& st) -> uint4 {
    return *(st.kin ? reinterpret_cast<const uint4*>(wt + ((size_t)st.t * a.Npad + j * 16 + (lane & 15)) * a.C + st.c)
                    : zero);
  };
  // set X holds the operands of the current step, set Y those of the next
  uint4 xa[RT], ya[RT], xb[NBP], yb[NBP];
  auto load = [&](uint4 (&sa)[RT], uint4 (&sb)[NBP], const Step& st) {
#pragma unroll
    for (int i = 0; i < RT; ++i) sa[i] = ld_a(i, st);
    if constexpr (PB) {
#pragma unroll
      for (int j = 0; j < NB; ++j) sb[j] = ld_b(j, st);
    }
  };
  auto mma = [&](const uint4 (&sa)[RT], const uint4 (&sb)[NBP], const Step& st) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bf16x8 bv = __builtin_bit_cast(bf16x8, PB ? sb[j] : ld_b(j, st));
#pragma unroll
      for (int i = 0; i < RT; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, sa[i]), bv, acc[i][j], 0, 0, 0);
    }
  };
  Step cur{kq / a.C, kq - (kq / a.C) * a.C, kq < K};
  load(xa, xb, cur);
  // two steps per trip; a trailing step past K reads zeros and adds nothing
  for (int k0 = 0; k0 < K; k0 += 64) {
    const Step s1 = next(cur);
    load(ya, yb, s1);
    mma(xa, xb, cur);
    const Step s2 = next(s1);
    load(xa, xb, s2);
    mma(ya, yb, s1);
    cur = s2;
  }
  // epilogue: rows 4 (lane / 16) + i of each row tile, column 16 j + lane % 16
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = j * 16 + (lane & 15);
      if (n >= a.N) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const long r = row0 + rt * 16 + (lane >> 4) * 4 + i;
        if (r >= nrows) continue;
        const bool on = a.mask == nullptr || bf2f(a.mask[(size_t)r * a.N + n]) > 0.f;
        a.dst[(size_t)r * a.N + n] = on ? f2bf(acc[rt][j][i]) : (uint16_t)0;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// 3x3x3 layers.  A block's rows are a 16 x 4 x RT box of output voxels (x
// fastest; wavefront w takes y0 + w % 4, MFMA column m takes x0 + m, row tile i
// takes z0 + i); NH = 2 puts two wavefronts on a row, each with its own NT
// column tiles of 16 output channels.  The input box with its one-voxel halo
// (zeros outside the grid) is staged in LDS once, all C channels, and every tap
// reads its operand there at a fixed offset.  The block marches along z: the
// next box is loaded into registers while the MFMAs of this one run where its
// LDS leaves one block per CU; below that the other blocks of the CU hide the
// loads.  Weights stay in registers for the whole march where they are at most
// 28 fragments (C <= 32 at NT = 1), else each tap's are loaded two taps ahead.  Voxels of 32 channels and more are padded by 16 bytes in LDS, so that
// the eight voxels of one read phase fall into different banks.
//
// The MFMA takes the weights as its A operand, so a lane ends up with four
// consecutive output channels of one voxel and stores 8 bytes; the reduction
// runs over k = t C + c in steps of 32, taps first.
//
// Bound by LDS reads (1 KiB per NT MFMAs) and, at 16 channels, by HBM: the
// 16 -> 16 layer moves 64 B per voxel, 3.6 TB/s at 512 x 512 x 128.  Times at
// that volume, first with one box per block, 64-bit addresses formed per load
// and 2-byte stores (64 -> 32 and wider: gathered from global memory): 1 -> 16
// channels 1.08 -> 0.45 ms, 16 -> 16 1.59 -> 0.59, 32 -> 16 3.81 -> 1.04,
// 64 -> 32 (256 x 256 x 64) 2.32 -> 0.83, 128 -> 64 (128 x 128 x 32) 1.15 -> 0.75.
// ---------------------------------------------------------------------------
constexpr int kHbX = 18, kHbY = 6;  // halo box extent in x and y

template <int C>
__host__ __device__ constexpr int conv_stride() { return C >= 32 ? C + 8 : C; }  // elements per LDS voxel

template <int C, int NT, int NH, int RT, int MODE, bool IN32>
__global__ void __launch_bounds__(256 * NH, NH == 1 && (RT + 2) * 108 * conv_stride<C>() * 2 > 80 * 1024 ? 1 : 2)
k_conv3(ConvArgs a) {
  constexpr int BZ = RT + 2, NV = kHbX * kHbY * BZ, CCH = C / 8, VS = conv_stride<C>();
  constexpr int ZS = kHbY * kHbX * VS;                      // one plane of the box
  // threads and 16-byte chunks per voxel of one staging half, chunks per thread and plane
  constexpr int NTHR = 256 * NH, NTH = C > 8 ? NTHR / 2 : NTHR, CCT = C > 8 ? CCH / 2 : 1;
  constexpr int NCP = (kHbX * kHbY * CCT + NTH - 1) / NTH;
  constexpr int NSTEP = (27 * C + 31) / 32, KC = C >= 32 ? C / 32 : 1;
  constexpr bool PRE = NSTEP * NT <= 28;                    // weights in registers
  static_assert(PRE || C >= 32, "weights of several taps per step stay in registers");
  constexpr bool PF = NV * VS * 2 > 64 * 1024;              // one block per CU: next box prefetched
  __shared__ __align__(16) uint16_t s_box[NV * VS];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wy = wv & 3, nh = wv >> 2;
  const int lx = lane & 15, g = lane >> 4;
  // block -> (column group, x, y, z run): column groups share the input box
  uint32_t id = xcd_tile(blockIdx.x, gridDim.x);
  const int ngrp = a.Npad / (16 * NT * NH);
  const int n0 = ((int)(id % ngrp) * NH + nh) * NT * 16;
  id /= ngrp;
  const int xt = (a.W + 15) / 16, yt = (a.H + 3) / 4, zt = (a.D + RT - 1) / RT;
  const int x0 = (int)(id % xt) * 16;
  id /= xt;
  const int y0 = (int)(id % yt) * 4;
  const int zb = (int)(id / yt) * a.zrun, ze = min(zt, zb + a.zrun);

  // Staging: half of the wavefronts load channels [0, C/2) from src, the other
  // half [C/2, C) from src2 (all of them the one chunk of C = 8).  A thread's
  // chunks sit at the same offsets in every plane, computed once; the six rows
  // of a plane are a buffer descriptor, empty for planes outside the grid, and
  // chunks outside it in x or y take an offset past every one: both read 0.
  const uint32_t half = C > 8 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (NTHR / 2)) : 0u;
  const int th = (int)threadIdx.x - (int)half * (NTHR / 2);
  const uint32_t esz = IN32 ? 4u : (uint32_t)a.src_cs * 2u;   // bytes per source voxel
  const uint32_t rowb = (uint32_t)a.W * esz;
  uint32_t goff[NCP];
  int loff[NCP];   // LDS element offset, or -1
#pragma unroll
  for (int i = 0; i < NCP; ++i) {
    const int e = th + i * NTH, v = e / CCT, q = e % CCT;
    const int x = x0 + v % kHbX - 1, y = y0 + v / kHbX - 1;
    const bool in = e < kHbX * kHbY * CCT;
    goff[i] = in && (unsigned)x < (unsigned)a.W && (unsigned)y < (unsigned)a.H
                  ? (uint32_t)(v / kHbX) * rowb + x * esz + (IN32 ? 0u : q * 16u) : kBufOff;
    loff[i] = in ? v * VS + (int)(half * CCT + q) * 8 : -1;
  }
  const char* gsrc = IN32 ? reinterpret_cast<const char*>(a.src32)
                          : reinterpret_cast<const char*>(half ? a.src2 : a.src);
  u32x4 st[BZ][NCP];
  float st32[BZ][NCP];
  auto load_box = [&](int z0) {
#pragma unroll
    for (int b = 0; b < BZ; ++b) {
      const int z = z0 + b - 1;
      const __amdgpu_buffer_rsrc_t r =
          buf_rsrc(gsrc + ((long)z * a.H + y0 - 1) * rowb, (unsigned)z < (unsigned)a.D ? kHbY * rowb : 0u);
#pragma unroll
      for (int i = 0; i < NCP; ++i) {
        if constexpr (IN32) st32[b][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)goff[i], 0, 0));
        else st[b][i] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)goff[i], 0, 0);
      }
    }
  };
  auto store_box = [&]() {
#pragma unroll
    for (int i = 0; i < NCP; ++i) {
      if (loff[i] < 0) continue;
#pragma unroll
      for (int b = 0; b < BZ; ++b) {
        u32x4 v;
        if constexpr (IN32) v = u32x4{f2bf(a.scale * st32[b][i]), 0u, 0u, 0u};
        else v = st[b][i];
        *reinterpret_cast<u32x4*>(s_box + loff[i] + b * ZS) = v;
      }
    }
  };
  // weight fragment of the reduction elements k = 8 g .. 8 g + 7 of a step
  const uint16_t* wt = a.wt;
  auto ld_w = [&](int t, int c, int j) -> bf16x8 {
    const bool on = C >= 32 || t < 27;
    return __builtin_bit_cast(
        bf16x8, *(on ? reinterpret_cast<const u32x4*>(wt + ((size_t)t * a.Npad + n0 + j * 16 + lx) * C + c)
                     : reinterpret_cast<const u32x4*>(&g_gg_zero)));
  };
  // LDS element offset of tap t relative to this lane's voxel at (0, 0, 0)
  auto tap = [&](int t) -> int {
    const int dz = MODE == GG_CONV3_BWD ? 2 - t / 9 : t / 9, dy = MODE == GG_CONV3_BWD ? 2 - (t / 3) % 3 : (t / 3) % 3,
              dx = MODE == GG_CONV3_BWD ? 2 - t % 3 : t % 3;
    return ((dz * kHbY + dy) * kHbX + dx) * VS;
  };
  const uint16_t* lane_box = s_box + (wy * kHbX + lx) * VS + (C >= 32 ? g * 8 : (C == 16 ? (g & 1) * 8 : 0));

  // PRE: every fragment; else a ring of three taps, loaded two taps ahead
  bf16x8 wr[PRE ? NSTEP : 3 * KC][NT];
  if constexpr (PRE) {
#pragma unroll
    for (int k = 0; k < NSTEP; ++k)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if constexpr (C == 8) wr[k][j] = ld_w(4 * k + g, 0, j);
        else if constexpr (C == 16) wr[k][j] = ld_w(2 * k + (g >> 1), (g & 1) * 8, j);
        else wr[k][j] = ld_w(k / KC, (k % KC) * 32 + g * 8, j);
      }
  }
  auto ld_tap = [&](int t, int slot) {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int j = 0; j < NT; ++j) wr[PRE ? 0 : slot * KC + kc][j] = ld_w(t, kc * 32 + g * 8, j);
  };
  // output offsets of this lane's voxel and channels in the four rows of a
  // plane (kBufOff: not stored)
  const uint32_t drow = (uint32_t)a.W * a.dst_cs * 2u, mrow = (uint32_t)a.W * a.mask_cs * 2u;
  uint32_t doff[NT], doff2[NT], moff[NT];
  float bs[NT][4];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int x = x0 + lx, n = n0 + j * 16 + g * 4;
    const bool on = x < a.W && y0 + wy < a.H && n < a.N;
    const uint32_t o = wy * drow + (uint32_t)x * a.dst_cs * 2u;
    doff[j] = on && n < a.nsplit ? o + n * 2u : kBufOff;
    doff2[j] = on && n >= a.nsplit ? o + (n - a.nsplit) * 2u : kBufOff;
    moff[j] = on ? wy * mrow + ((uint32_t)x * a.mask_cs + n) * 2u : kBufOff;
#pragma unroll
    for (int r = 0; r < 4; ++r) bs[j][r] = a.bias && n < a.N ? a.bias[n + r] : 0.f;
  }
  if (PF && zb < ze) load_box(zb * RT);
  for (int zi = zb; zi < ze; ++zi) {
    const int z0 = zi * RT;
    if (!PF) load_box(z0);
    __syncthreads();   // the previous box has been read
    store_box();
    __syncthreads();
    if (PF && zi + 1 < ze) load_box(z0 + RT);
    f32x4 acc[RT][NT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (PRE) {
#pragma unroll
      for (int k = 0; k < NSTEP; ++k) {
        int off;
        bool in = true;   // the last step of C < 32 has taps past 26
        if constexpr (C >= 32) {
          off = tap(k);
        } else if constexpr (C == 16) {
          const int o0 = tap(2 * k), o1 = 2 * k + 1 < 27 ? tap(2 * k + 1) : 0;
          off = (g >> 1) ? o1 : o0;
          in = 2 * k + 1 < 27 || (g >> 1) == 0;
        } else {
          const int o0 = tap(4 * k), o1 = tap(4 * k + 1), o2 = tap(4 * k + 2), o3 = 4 * k + 3 < 27 ? tap(4 * k + 3) : 0;
          off = g < 2 ? (g == 0 ? o0 : o1) : (g == 2 ? o2 : o3);
          in = 4 * k + 3 < 27 || g < 3;
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          u32x4 raw = *reinterpret_cast<const u32x4*>(lane_box + off + i * ZS);
          if (C < 32 && k == NSTEP - 1 && !in) raw = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[k][j], __builtin_bit_cast(bf16x8, raw), acc[i][j], 0, 0, 0);
        }
      }
    } else {
      // a fresh pointer per box: the loads of all taps would otherwise be
      // hoisted out of the march into registers it does not have
      asm volatile("" : "+s"(wt));
      ld_tap(0, 0);
      ld_tap(1, 1);
#pragma unroll 1
      for (int dz = 0; dz < 3; ++dz) {
        const uint16_t* zbox = lane_box + (MODE == GG_CONV3_BWD ? 2 - dz : dz) * ZS;
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          ld_tap(min(dz * 9 + u + 2, 26), (u + 2) % 3);   // past the last tap: not used
          const int uu = MODE == GG_CONV3_BWD ? 8 - u : u;
          const int off = ((uu / 3) * kHbX + uu % 3) * VS;
#pragma unroll
          for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
            for (int i = 0; i < RT; ++i) {
              const bf16x8 xv = *reinterpret_cast<const bf16x8*>(zbox + off + i * ZS + kc * 32);
#pragma unroll
              for (int j = 0; j < NT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[(u % 3) * KC + kc][j], xv, acc[i][j], 0, 0, 0);
            }
          }
        }
      }
    }
    // D row 4 g + r is an output channel, column lx a voxel
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int z = z0 + i;
        if (z >= a.D) break;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = acc[i][j][r];
          if (a.bias) v[r] += bs[j][r];
          if (a.relu) v[r] = fmaxf(v[r], 0.f);
        }
        u32x2 o = {bf_pack(v[0], v[1]), bf_pack(v[2], v[3])};
        if (a.mask) {
          const __amdgpu_buffer_rsrc_t rm =
              buf_rsrc(reinterpret_cast<const char*>(a.mask) + ((long)z * a.H + y0) * mrow, 4 * mrow);
          o = bf_mask(o, __builtin_amdgcn_raw_buffer_load_b64(rm, (int)moff[j], 0, 0));
        }
        const long row = ((long)z * a.H + y0) * drow;
        if (n0 + j * 16 < a.nsplit)
          __builtin_amdgcn_raw_buffer_store_b64(o, buf_rsrc(reinterpret_cast<char*>(a.dst) + row, 4 * drow),
                                                (int)doff[j], 0, 0);
        if (n0 + j * 16 + 16 > a.nsplit)
          __builtin_amdgcn_raw_buffer_store_b64(o, buf_rsrc(reinterpret_cast<char*>(a.dst2) + row, 4 * drow),
                                                (int)doff2[j], 0, 0);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradient: dW[t][c][n] = sum_r S(r + offset(t))[c] G(r)[n], and the bias
// gradient sum_r G(r)[n] from the same pass ([t][c][n] is the [tap][cin][cout]
// layout of the master weights).
//
// A block takes a run of 16 x 4 x 4 boxes of rows.  It stages a box of G and
// the box of S with its one-voxel halo (zeros outside the grid) in LDS once,
// channels-last as they lie in memory, and every tap then takes its operand
// from there at a shifted voxel; the 16-bit transposing LDS read turns four
// rows of 16 channels into the 8 reduction (row) elements per lane the MFMA
// wants.  A wavefront owns one 16 x 16 (n, c) tile of every tap (27 x 4
// accumulators); a block covers up to 2 x 2 such tiles, or splits the box's
// rows over its wavefronts when the layer has fewer, and adds their sums
// through LDS at the end.  Each block writes one partial; k_finish_grads adds
// the partials in order, so the result is the same on every run.
// The pass is bound by those LDS reads (1 KiB per MFMA).  Staging S per tap
// from global memory with 2-byte transposes, and summing the bias with one
// thread per channel, took 13 ms of a 15.07 ms training step at 64 x 64 x 32
// (levels 4, base 16); with this kernel the step takes 2.15 ms.
// ---------------------------------------------------------------------------
constexpr int kWgBX = 16, kWgBY = 4, kWgBZ = 4;   // rows of a box: 8 slabs of 32
constexpr int kWgRows = kWgBX * kWgBY * kWgBZ;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// Element offset of an LDS voxel: CS channels and 16 bytes of padding, so that
// the rows a transposing read gathers fall into different banks.
template <int CS>
__host__ __device__ constexpr int wg_stride() { return CS + 8; }

__device__ __forceinline__ s16x4 lds_tr(const uint16_t* p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(const __attribute__((address_space(3))) uint16_t*)p);
}

// TAPS: 27 (3x3x3, S with halo) or 1 (1x1x1 layers, and one tap of an
// up-convolution per blockIdx.z: G at the fine voxel 2q + tap).  CT x NT: the
// 16-channel tiles of S and G a block covers.
template <int TAPS, int CT, int NT>
__global__ void __launch_bounds__(256) k_wgrad(WgradArgs a) {
  constexpr bool CONV = TAPS == 27;
  constexpr int PB = CT * NT, RP = 4 / PB;       // tiles per block, row parts per tile
  constexpr int HX = CONV ? kWgBX + 2 : kWgBX, HY = CONV ? kWgBY + 2 : kWgBY, HZ = CONV ? kWgBZ + 2 : kWgBZ;
  constexpr int SS = wg_stride<CT * 16>(), SG = wg_stride<NT * 16>();
  constexpr int NSV = HX * HY * HZ;
  constexpr int PIECE = CONV ? 9 : 1;             // taps reduced over the row parts at a time
  constexpr int kStage = (NSV * SS + kWgRows * SG) * 2, kRed = 4 * PIECE * 64 * 16;
  __shared__ __align__(16) unsigned char s_raw[kStage > kRed ? kStage : kRed];
  uint16_t* ss = reinterpret_cast<uint16_t*>(s_raw);
  uint16_t* sg = ss + NSV * SS;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int pair = wv % PB, rp = wv / PB;
  const int cg = (a.Cpad / 16) / CT;              // channel groups of S
  const int c0 = (blockIdx.y % cg) * CT * 16, n0 = (blockIdx.y / cg) * NT * 16;
  const int ci = pair % CT, ni = pair / CT;
  const int tap = a.mode == GG_UP_FWD ? (int)blockIdx.z : 0;
  const int bxn = (a.W + kWgBX - 1) / kWgBX, byn = (a.H + kWgBY - 1) / kWgBY, bzn = (a.D + kWgBZ - 1) / kWgBZ;
  const int nbox = bxn * byn * bzn;
  const int b0 = (int)((long)blockIdx.x * nbox / gridDim.x), b1 = (int)((long)(blockIdx.x + 1) * nbox / gridDim.x);
  f32x4 acc[TAPS], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < TAPS; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // transposing read: lane i of a group of 16 supplies row i / 4, channels 4 (i % 4)
  const int tr = (lane & 15) >> 2, tq = (lane & 3) * 4, kg = lane >> 4;
  const bf16x8 ones = __builtin_bit_cast(bf16x8, (s16x8)(short)0x3f80);
  for (int b = b0; b < b1; ++b) {
    const int x0 = (b % bxn) * kWgBX, y0 = ((b / bxn) % byn) * kWgBY, z0 = (b / (bxn * byn)) * kWgBZ;
    __syncthreads();
    for (int e = threadIdx.x; e < NSV * CT * 2; e += 256) {
      const int v = e / (CT * 2), q = e % (CT * 2);
      constexpr int O = CONV ? 1 : 0;
      const int x = x0 + v % HX - O, y = y0 + (v / HX) % HY - O, z = z0 + v / (HX * HY) - O, c = c0 + q * 8;
      const bool on = (unsigned)x < (unsigned)a.W && (unsigned)y < (unsigned)a.H && (unsigned)z < (unsigned)a.D && c < a.C;
      const long vox = ((long)z * a.H + y) * a.W + x;
      uint4 val;
      if (a.s32) val = make_uint4(on ? f2bf(a.scale * a.s32[vox]) : 0u, 0u, 0u, 0u);
      else val = *(on ? reinterpret_cast<const uint4*>((c < a.ssplit ? a.s : a.s2) + vox * a.s_cs + c) : &g_gg_zero);
      *reinterpret_cast<uint4*>(ss + v * SS + q * 8) = val;
    }
    for (int e = threadIdx.x; e < kWgRows * NT * 2; e += 256) {
      const int v = e / (NT * 2), q = e % (NT * 2);
      const int x = x0 + v % kWgBX, y = y0 + (v / kWgBX) % kWgBY, z = z0 + v / (kWgBX * kWgBY), n = n0 + q * 8;
      const bool on = x < a.W && y < a.H && z < a.D && n < a.N;
      long gv = ((long)z * a.H + y) * a.W + x;
      if (a.mode == GG_UP_FWD)
        gv = ((long)(2 * z + (tap >> 2)) * (2 * a.H) + 2 * y + ((tap >> 1) & 1)) * (2 * a.W) + 2 * x + (tap & 1);
      const uint4 val = *(on ? reinterpret_cast<const uint4*>(a.g + gv * a.g_cs + n) : &g_gg_zero);
      *reinterpret_cast<uint4*>(sg + v * SG + q * 8) = val;
    }
    __syncthreads();
    // slab k of 32 rows: y rows 2 (k % 2), 2 (k % 2) + 1 of plane k / 2; this
    // lane's 8 rows are x = 8 (kg % 2) .. + 7 of row kg / 2
    for (int k = rp; k < kWgRows / 32; k += RP) {
      const int yy = (k & 1) * 2 + (kg >> 1), zz = k >> 1, xx = (kg & 1) * 8 + tr;
      auto frag = [&](const uint16_t* base, int stride) {
        const s16x4 lo = lds_tr(base), hi = lds_tr(base + 4 * stride);
        s16x8 f;
        f[0] = lo[0]; f[1] = lo[1]; f[2] = lo[2]; f[3] = lo[3];
        f[4] = hi[0]; f[5] = hi[1]; f[6] = hi[2]; f[7] = hi[3];
        return __builtin_bit_cast(bf16x8, f);
      };
      const bf16x8 gf = frag(sg + ((zz * kWgBY + yy) * kWgBX + xx) * SG + ni * 16 + tq, SG);
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf, ones, accb, 0, 0, 0);
      const uint16_t* sb = ss + ((zz * HY + yy) * HX + xx) * SS + ci * 16 + tq;
#pragma unroll
      for (int t = 0; t < TAPS; ++t) {
        const int o = CONV ? ((t / 9) * HY + (t / 3) % 3) * HX + t % 3 : 0;
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf, frag(sb + o * SS, SS), acc[t], 0, 0, 0);
      }
    }
  }
  // D rows n = 4 (lane / 16) + i, columns c = lane % 16; the row parts of a
  // tile are added in order
  const int c = c0 + ci * 16 + (lane & 15), n = n0 + ni * 16 + (lane >> 4) * 4;
  const size_t count = (size_t)a.taps * a.C * a.N;
  float* part = a.part + (size_t)blockIdx.x * count;
  auto store = [&](int t, f32x4 v) {
    if (c >= a.C) return;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) part[((size_t)t * a.C + c) * a.N + n + i] = v[i];
  };
  auto store_bias = [&](f32x4 v) {
    if (blockIdx.y % cg != 0 || ci != 0 || (lane & 15) != 0) return;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n + i < a.N) a.bpart[((size_t)blockIdx.x * gridDim.z + blockIdx.z) * a.N + n + i] = v[i];
  };
  if constexpr (RP == 1) {
#pragma unroll
    for (int t = 0; t < TAPS; ++t) store(CONV ? t : tap, acc[t]);
    store_bias(accb);
  } else {
    f32x4* red = reinterpret_cast<f32x4*>(s_raw);   // [4 waves][PIECE][64]
#pragma unroll
    for (int p = 0; p < TAPS / PIECE; ++p) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PIECE; ++j) red[(wv * PIECE + j) * 64 + lane] = acc[p * PIECE + j];
      __syncthreads();
      for (int j = rp; j < PIECE; j += RP) {
        f32x4 v = red[(pair * PIECE + j) * 64 + lane];
#pragma unroll
        for (int r = 1; r < RP; ++r) v += red[((r * PB + pair) * PIECE + j) * 64 + lane];
        store(CONV ? p * PIECE + j : tap, v);
      }
    }
    __syncthreads();
    red[wv * 64 + lane] = accb;
    __syncthreads();
    if (rp == 0) {
#pragma unroll
      for (int r = 1; r < RP; ++r) accb += red[(r * PB + pair) * 64 + lane];
      store_bias(accb);
    }
  }
}

// Gradients from their partials (weights, biases and the loss are table
// entries): out[e] = sum over b of part[b * count + e].  A block takes 64
// elements; its four groups of 64 threads add a quarter of the partials each,
// in order, and the quarters are added in order, so every run gives the same
// bits.  With lr > 0 the same thread applies Adam to its parameter (a1 = 1 -
// b1, a2 = 1 - b2 and the bias corrections c1, c2 come from the host in FP64;
// 1 - 0.999f in FP32 is off by 5e-5 relative).
__global__ void __launch_bounds__(256) k_finish_grads(GradTable tab, AdamArgs ad) {
  __shared__ float s_q[4][64];
  int k = 0;
  while (k + 1 < tab.n && (int)blockIdx.x >= tab.e[k + 1].block0) ++k;
  const GradEntry g = tab.e[k];
  const int t = threadIdx.x & 63, q = threadIdx.x >> 6;
  const long e = (long)((int)blockIdx.x - g.block0) * 64 + t;
  const int p0 = (int)((long)q * g.parts / 4), p1 = (int)((long)(q + 1) * g.parts / 4);
  float s = 0.f;
  if (e < g.count) {
    const float* src = g.part + e;
#pragma unroll 8
    for (int b = p0; b < p1; ++b) s += src[(size_t)b * g.count];
  }
  s_q[q][t] = s;
  __syncthreads();
  if (q != 0 || e >= g.count) return;
  const float gi = s_q[0][t] + s_q[1][t] + s_q[2][t] + s_q[3][t];
  g.out[e] = gi;
  if (g.param < 0 || !(ad.lr > 0.f)) return;
  const size_t i = (size_t)g.param + e;
  const float mi = ad.b1 * ad.m[i] + ad.a1 * gi;
  const float vi = ad.b2 * ad.v[i] + ad.a2 * gi * gi;
  ad.m[i] = mi;
  ad.v[i] = vi;
  ad.w[i] -= ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
}

// ---------------------------------------------------------------------------
// Up-convolution (2x2x2, stride 2): the coarse voxels times [cu] x [8 c]
// weights; column d c + co is channel co of the fine voxel 2 q + d.  A
// wavefront takes 64 coarse voxels and every column tile (or the share of
// blockIdx.y); the weights are the MFMA's A operand, so a lane stores four
// channels of one fine voxel.  Bound by the stores: 16 c bytes per coarse voxel,
// whole lines as the skip connection lies in a buffer of its own (32 -> 16
// channels at 512 x 512 x 128: 1.60 ms with 2-byte stores into half of each
// voxel's line, now 0.55, 4.3 TB/s of stores and loads).
// ---------------------------------------------------------------------------
template <int KS>
__global__ void __launch_bounds__(256) k_up_fwd(UpArgs a) {
  const int lane = threadIdx.x & 63, lx = lane & 15, g = lane >> 4;
  const long nrows = (long)a.D * a.H * a.W;
  const long r0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  bf16x8 xv[4][KS];
  long fv[4];   // fine voxel 2 q of each tile's column, or -1
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const long r = r0 + i * 16 + lx;
    const bool on = r < nrows;   // nrows < 2^31
    const uint32_t zy = (uint32_t)r / (uint32_t)a.W, x = (uint32_t)r - zy * a.W, z = zy / (uint32_t)a.H, y = zy - z * a.H;
    fv[i] = on ? ((long)(2 * z) * (2 * a.H) + 2 * y) * (2 * a.W) + 2 * x : -1;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int c = k * 32 + g * 8;
      xv[i][k] = __builtin_bit_cast(
          bf16x8, on && c < a.cu ? *reinterpret_cast<const u32x4*>(a.src + r * a.cu + c) : zero);
    }
  }
  const int tiles = 8 * a.c / 16, per = tiles / (int)gridDim.y, j0 = (int)blockIdx.y * per;
  auto ld_w = [&](int j, int k) {
    const int c = k * 32 + g * 8;
    return __builtin_bit_cast(
        bf16x8, c < a.cu ? *reinterpret_cast<const u32x4*>(a.wt + ((size_t)j * 16 + lx) * a.cu + c) : zero);
  };
  bf16x8 wn[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) wn[k] = ld_w(j0, k);
  for (int j = j0; j < j0 + per; ++j) {
    bf16x8 w[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      w[k] = wn[k];
      wn[k] = ld_w(min(j + 1, tiles - 1), k);
    }
    const int n = j * 16 + g * 4, d = n / a.c, co = n - d * a.c;
    float b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r] = a.bias[co + r];
    const long off = ((long)(d >> 2) * (2 * a.H) + ((d >> 1) & 1)) * (2 * a.W) + (d & 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k], xv[i][k], acc, 0, 0, 0);
      if (fv[i] >= 0)
        *reinterpret_cast<u32x2*>(a.dst + (fv[i] + off) * a.c + co) =
            u32x2{bf_pack(acc[0] + b[0], acc[1] + b[1]), bf_pack(acc[2] + b[2], acc[3] + b[3])};
    }
  }
}

// Head (1x1x1, one output channel, FP32): row 0 of the weight operand is real.
template <int KS>
__global__ void __launch_bounds__(256) k_head(const uint16_t* __restrict__ src, int C, const uint16_t* __restrict__ wt,
                                              const float* bias, int relu, float* __restrict__ out, long nvox) {
  const int lane = threadIdx.x & 63, lx = lane & 15, g = lane >> 4;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  bf16x8 w[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const int c = k * 32 + g * 8;
    w[k] = __builtin_bit_cast(bf16x8, c < C ? *reinterpret_cast<const u32x4*>(wt + (size_t)lx * C + c) : zero);
  }
  const float b = bias[0];
  for (long r0 = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64; r0 < nvox; r0 += (long)gridDim.x * 256) {
    u32x4 xv[4][KS];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const long r = r0 + i * 16 + lx;
        const int c = k * 32 + g * 8;
        xv[i][k] = r < nvox && c < C ? *reinterpret_cast<const u32x4*>(src + r * C + c) : zero;
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KS; ++k)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k], __builtin_bit_cast(bf16x8, xv[i][k]), acc, 0, 0, 0);
      const long r = r0 + i * 16 + lx;
      const float v = acc[0] + b;
      if (g == 0 && r < nvox) out[r] = relu ? fmaxf(v, 0.f) : v;
    }
  }
}

// ---------------------------------------------------------------------------
// Max pooling 2x2x2, eight channels per thread (C is a multiple of 8, channels
// contiguous).  Forward: the first largest value of the window and, for
// training, its index.
// ---------------------------------------------------------------------------
// f(coarse voxel, first fine voxel of its window, channel) for every coarse
// voxel and chunk of 8 channels: x and channels over blockIdx.x, rows and planes
// over blockIdx.y and .z
template <class F>
__device__ __forceinline__ void for_pool(int C, int D, int H, int W, F f) {
  const uint32_t cc = (uint32_t)C / 8, e = blockIdx.x * 256u + threadIdx.x, x = e / cc;
  if (x >= (uint32_t)W) return;
  for (int z = blockIdx.z; z < D; z += gridDim.z)
    for (int y = blockIdx.y; y < H; y += gridDim.y)
      f(((long)z * H + y) * W + x, ((long)(2 * z) * (2 * H) + 2 * y) * (2 * W) + 2 * x, (int)(e - x * cc) * 8);
}

__global__ void __launch_bounds__(256) k_pool_fwd(const uint16_t* __restrict__ x, uint16_t* __restrict__ y,
                                                  uint8_t* __restrict__ idx, int C, int D, int H, int W) {
  for_pool(C, D, H, W, [&](long q, long f0, int c) {
    u32x4 v[8];
#pragma unroll
    for (int d = 0; d < 8; ++d)
      v[d] = *reinterpret_cast<const u32x4*>(x + (f0 + ((long)(d >> 2) * (2 * H) + ((d >> 1) & 1)) * (2 * W) + (d & 1)) * C + c);
    u32x4 best = v[0], bi = {0u, 0u, 0u, 0u};   // bi: per channel the index, 16 bits each
#pragma unroll
    for (int d = 1; d < 8; ++d)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t b = best[k], w = v[d][k];
        const bool lo = __uint_as_float(w << 16) > __uint_as_float(b << 16);
        const bool hi = __uint_as_float(w & 0xffff0000u) > __uint_as_float(b & 0xffff0000u);
        best[k] = (lo ? w & 0xffffu : b & 0xffffu) | (hi ? w & 0xffff0000u : b & 0xffff0000u);
        bi[k] = (lo ? (uint32_t)d : bi[k] & 0xffffu) | (hi ? (uint32_t)d << 16 : bi[k] & 0xffff0000u);
      }
    *reinterpret_cast<u32x4*>(y + q * C + c) = best;
    if (idx != nullptr) {
      u32x2 o;
#pragma unroll
      for (int k = 0; k < 2; ++k)
        o[k] = (bi[2 * k] & 7u) | ((bi[2 * k] >> 16) << 8) | ((bi[2 * k + 1] & 7u) << 16) | ((bi[2 * k + 1] >> 16) << 24);
      *reinterpret_cast<u32x2*>(idx + q * C + c) = o;
    }
  });
}

// Backward, onto the gradient that came through the skip connection: g at the
// window's winner grows by the pooled gradient (rounded), and the ReLU of the
// pooled layer (y) masks every voxel.
__global__ void __launch_bounds__(256) k_pool_bwd(const uint16_t* __restrict__ gy, const uint8_t* __restrict__ idx,
                                                  const uint16_t* __restrict__ y, uint16_t* __restrict__ g, int C,
                                                  int D, int H, int W) {
  for_pool(C, D, H, W, [&](long q, long f0, int c) {
    const u32x4 gv = *reinterpret_cast<const u32x4*>(gy + q * C + c);
    const u32x2 iv = *reinterpret_cast<const u32x2*>(idx + q * C + c);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const long o = (f0 + ((long)(d >> 2) * (2 * H) + ((d >> 1) & 1)) * (2 * W) + (d & 1)) * C + c;
      const u32x4 yv = *reinterpret_cast<const u32x4*>(y + o);
      u32x4 gg = *reinterpret_cast<const u32x4*>(g + o);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float r[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t w = (iv[k >> 1] >> (16 * (k & 1) + 8 * h)) & 0xffu;
          const float a = bf2f((uint16_t)(gg[k] >> (16 * h))), b = bf2f((uint16_t)(gv[k] >> (16 * h)));
          r[h] = w == (uint32_t)d ? a + b : a;
          if (!(bf2f((uint16_t)(yv[k] >> (16 * h))) > 0.f)) r[h] = 0.f;
        }
        gg[k] = bf_pack(r[0], r[1]);
      }
      *reinterpret_cast<u32x4*>(g + o) = gg;
    }
  });
}

// Weighted MSE of the head's pre-activation y (FP32) against t, weight pos_w
// where t > 0 and 1 elsewhere; gradient 2 w (y - t) / n into channel 0 of g[v][8], zeros in the others
__global__ void k_mse(const float* y, const float* t, long n, float inv_n, float pos_w, uint16_t* g, float* loss) {
  __shared__ float red[4];
  float s = 0.f;
  for (long v = (long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (long)gridDim.x * blockDim.x) {
    const float d = y[v] - t[v];
    const float w = t[v] > 0.f ? pos_w : 1.f;
    s += w * d * d;
    *reinterpret_cast<u32x4*>(g + v * 8) = u32x4{f2bf(2.f * w * d * inv_n), 0u, 0u, 0u};
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) loss[blockIdx.x] = (red[0] + red[1] + red[2] + red[3]) * inv_n;   // per-block partial
}

// Pack FP32 master weights W[t][cin][cout] into BF16 B[t][n][c], every layer
// and use in one launch (a table entry each).  kind 1: n = cout, c = cin
// (forward); 0: n = cin, c = cout (input gradient); 2, the up-convolution
// forward: one tap, n = t cout + co, c = cin.  Channels beyond the real counts
// are zero.
__global__ void __launch_bounds__(256) k_pack(PackTable tab) {
  int k = 0;
  while (k + 1 < tab.n && (int)blockIdx.x >= tab.e[k + 1].block0) ++k;
  const PackEntry p = tab.e[k];
  const uint32_t e = (blockIdx.x - (uint32_t)p.block0) * 256u + threadIdx.x;
  if (e >= (uint32_t)p.T * p.Npad * p.Cpad) return;
  const uint32_t c = e % p.Cpad, r = e / p.Cpad, nn = r % p.Npad, t = r / p.Npad;
  float v = 0.f;
  if (p.kind == 1) {
    if (nn < (uint32_t)p.cout && c < (uint32_t)p.cin) v = p.w[(t * p.cin + c) * p.cout + nn];
  } else if (p.kind == 0) {
    if (nn < (uint32_t)p.cin && c < (uint32_t)p.cout) v = p.w[(t * p.cin + nn) * p.cout + c];
  } else {
    v = p.w[((nn / p.cout) * p.cin + c) * p.cout + nn % p.cout];
  }
  p.out[e] = f2bf(v);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static int ew_grid(size_t n) {
  size_t b = (n + 255) / 256;
  return (int)(b > 16384 ? 16384 : (b == 0 ? 1 : b));
}

// Blocks and z run of a 3x3x3 layer.  Big grids take boxes of RT planes and
// march along z in runs that leave about 2048 blocks.  Where the weights are
// streamed (64 channels and more) the box is as high as LDS allows, as each
// fragment then serves more rows: 64 -> 32 at 256 x 256 x 64 1.11 ms with 4 planes,
// 0.83 with 8 (1.71 with 2); 64 -> 64 0.30 -> 0.19; 128 -> 64 at 128 x 128 x 32 0.97
// with 2, 0.75 with 3.  Where they stay in registers (32 -> 16) 4 planes leave
// three blocks a unit: 1.09 ms, 1.38 with 5, 1.49 with 8; grids of fewer boxes than
// compute units (the coarse levels of a training crop) take one plane and 16
// output channels per block, which spreads them over more of the chip.
template <int C, int NT, int NH, int RT, bool IN32>
static hipError_t launch_conv3_t(ConvArgs a, hipStream_t s) {
  const long xy = (long)((a.W + 15) / 16) * ((a.H + 3) / 4), zt = (a.D + RT - 1) / RT;
  const long groups = a.Npad / (16 * NT * NH);
  a.zrun = (int)std::max<long>(1, std::min<long>(zt, xy * zt * groups / 2048));
  const dim3 g((unsigned)(xy * groups * ((zt + a.zrun - 1) / a.zrun)));
  if constexpr (!IN32) {
    if (a.bwd) {
      hipLaunchKernelGGL((k_conv3<C, NT, NH, RT, GG_CONV3_BWD, false>), g, dim3(256 * NH), 0, s, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_conv3<C, NT, NH, RT, GG_CONV3_FWD, IN32>), g, dim3(256 * NH), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_conv3(ConvArgs a, hipStream_t s) {
  if (a.N % 8 || a.Npad % 16 || a.src_cs % 8 || a.dst_cs % 4 || a.mask_cs % 4 || (a.src32 && (a.bwd || a.C != 8)))
    return hipErrorInvalidValue;
  // six rows of a plane are addressed with 31 bits
  if ((double)a.W * std::max(a.src_cs, std::max(a.dst_cs, a.mask_cs)) * 2 * kHbY >= 2147483648.0) return hipErrorInvalidValue;
  const int nt = a.Npad / 16;
  const bool in32 = a.src32 != nullptr;
  const int rt = a.C <= 64 ? 4 : 2;
  const long boxes = (long)((a.W + 15) / 16) * ((a.H + 3) / 4) * ((a.D + rt - 1) / rt) * ((nt + 3) / 4);
  const bool small = boxes < 256;
  if (in32) {
    if (small || nt == 1) return small ? launch_conv3_t<8, 1, 1, 1, true>(a, s) : launch_conv3_t<8, 1, 1, 8, true>(a, s);
    return nt == 2 ? launch_conv3_t<8, 2, 1, 4, true>(a, s) : launch_conv3_t<8, 2, 2, 4, true>(a, s);
  }
  switch (a.C) {
    case 8: return small || nt > 1 ? launch_conv3_t<8, 1, 1, 1, false>(a, s) : launch_conv3_t<8, 1, 1, 4, false>(a, s);
    case 16:
      if (!small && nt == 1) return launch_conv3_t<16, 1, 1, 4, false>(a, s);
      if (!small && nt == 2) return launch_conv3_t<16, 2, 1, 8, false>(a, s);
      return launch_conv3_t<16, 1, 1, 1, false>(a, s);
    case 32:
      if (!small && nt == 1) return launch_conv3_t<32, 1, 1, 4, false>(a, s);
      if (!small && nt == 2) return launch_conv3_t<32, 2, 1, 4, false>(a, s);
      if (!small && nt % 4 == 0) return launch_conv3_t<32, 2, 2, 4, false>(a, s);
      return launch_conv3_t<32, 1, 1, 1, false>(a, s);
    case 64:
      if (!small && nt == 2) return launch_conv3_t<64, 2, 1, 8, false>(a, s);
      if (!small && nt % 4 == 0) return launch_conv3_t<64, 2, 2, 8, false>(a, s);
      return launch_conv3_t<64, 1, 1, 1, false>(a, s);
    case 128:
      if (!small && nt % 4 == 0) return launch_conv3_t<128, 2, 2, 3, false>(a, s);
      return launch_conv3_t<128, 1, 1, 1, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gather_gemm(const GatherGemmArgs& a, hipStream_t s) {
  const long nrows = (long)a.D * a.H * a.W;
  if (nrows >= (1l << 31)) return hipErrorInvalidValue;
  // row tiles per wave: enough MFMAs per loaded fragment without exceeding the
  // accumulator budget (RT * NB <= 8 tiles of 16 x 16)
  auto grid = [&](int rt) { return dim3((unsigned)((nrows + 64 * rt - 1) / (64 * rt))); };
  auto by_mode = [&](auto nb, auto rt) -> hipError_t {
    constexpr int NB = decltype(nb)::value, RT = decltype(rt)::value;
    const dim3 g = grid(RT);
    switch (a.mode) {
      case GG_UP_BWD: hipLaunchKernelGGL((k_gather_gemm<NB, RT, GG_UP_BWD>), g, dim3(256), 0, s, a); break;
      case GG_POINT: hipLaunchKernelGGL((k_gather_gemm<NB, RT, GG_POINT>), g, dim3(256), 0, s, a); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  switch (a.Npad / 16) {
    case 1: return by_mode(I1{}, I4{});
    case 2: return by_mode(I2{}, I4{});
    case 4: return by_mode(I4{}, I2{});
    case 8: return by_mode(std::integral_constant<int, 8>{}, I1{});
    default: return hipErrorInvalidValue;
  }
}

int wgrad_blocks(int mode, int D, int H, int W, int N, int C) {
  const int nbox = ((W + kWgBX - 1) / kWgBX) * ((H + kWgBY - 1) / kWgBY) * ((D + kWgBZ - 1) / kWgBZ);
  const int tn = (N + 15) / 16, tc = (C + 15) / 16;
  const int groups = std::max(1, tn / 2) * std::max(1, tc / 2) * (mode == GG_UP_FWD ? 8 : 1);
  // about two blocks per compute unit; a block sums at least one box
  return std::min(nbox, std::max(1, 512 / groups > 256 ? 256 : 512 / groups));
}

hipError_t launch_wgrad(WgradArgs a, int blocks, hipStream_t s) {
  if (a.N < 1 || a.C < 1 || a.s_cs % 8 || a.ssplit % 8 || a.g_cs % 8 || (a.s32 && a.C != 1)) return hipErrorInvalidValue;
  const int tn = (a.N + 15) / 16, tc = (a.C + 15) / 16;
  if ((tn & (tn - 1)) || (tc & (tc - 1))) return hipErrorInvalidValue;
  a.Cpad = tc * 16;
  const int NT = tn > 1 ? 2 : 1, CT = tc > 1 ? 2 : 1;
  const bool conv = a.mode == GG_CONV3_FWD;
  a.taps = conv ? 27 : (a.mode == GG_UP_FWD ? 8 : 1);
  const dim3 g((unsigned)blocks, (unsigned)((tn / NT) * (tc / CT)), a.mode == GG_UP_FWD ? 8 : 1);
#define RIHVR_WG(CT_, NT_)                                                                \
  if (conv) hipLaunchKernelGGL((k_wgrad<27, CT_, NT_>), g, dim3(256), 0, s, a);           \
  else hipLaunchKernelGGL((k_wgrad<1, CT_, NT_>), g, dim3(256), 0, s, a);
  if (CT == 2 && NT == 2) { RIHVR_WG(2, 2) }
  else if (CT == 2) { RIHVR_WG(2, 1) }
  else if (NT == 2) { RIHVR_WG(1, 2) }
  else { RIHVR_WG(1, 1) }
#undef RIHVR_WG
  return hipGetLastError();
}

hipError_t launch_finish_grads(GradTable& tab, const AdamArgs& ad, hipStream_t s) {
  int blocks = 0;
  for (int k = 0; k < tab.n; ++k) {
    tab.e[k].block0 = blocks;
    blocks += (int)((tab.e[k].count + 63) / 64);
  }
  hipLaunchKernelGGL(k_finish_grads, dim3(blocks), dim3(256), 0, s, tab, ad);
  return hipGetLastError();
}

static dim3 pool_grid(int C, int D, int H, int W) {
  return dim3((unsigned)(((long)W * (C / 8) + 255) / 256), (unsigned)std::min(H, 65535), (unsigned)std::min(D, 65535));
}

hipError_t launch_pool_fwd(const uint16_t* x, uint16_t* y, uint8_t* idx, int C, int D, int H, int W, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_fwd, pool_grid(C, D, H, W), dim3(256), 0, s, x, y, idx, C, D, H, W);
  return hipGetLastError();
}

hipError_t launch_pool_bwd(const uint16_t* gy, const uint8_t* idx, const uint16_t* y, uint16_t* g, int C, int D, int H,
                           int W, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_bwd, pool_grid(C, D, H, W), dim3(256), 0, s, gy, idx, y, g, C, D, H, W);
  return hipGetLastError();
}

hipError_t launch_up_fwd(const UpArgs& a, hipStream_t s) {
  const long nrows = (long)a.D * a.H * a.W;
  if (nrows >= (1l << 31)) return hipErrorInvalidValue;
  const unsigned gx = (unsigned)((nrows + 255) / 256);
  // few coarse voxels: the column tiles are shared out so that more blocks run
  unsigned gy = 1;
  while (gx * gy < 512 && gy < (unsigned)a.c / 2) gy *= 2;
  const dim3 g(gx, gy);
  switch (a.cu) {
    case 16:
    case 32: hipLaunchKernelGGL(k_up_fwd<1>, g, dim3(256), 0, s, a); break;
    case 64: hipLaunchKernelGGL(k_up_fwd<2>, g, dim3(256), 0, s, a); break;
    case 128: hipLaunchKernelGGL(k_up_fwd<4>, g, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_head(const uint16_t* src, int C, const uint16_t* wt, const float* bias, int relu, float* out, long n,
                       hipStream_t s) {
  const dim3 g((unsigned)std::min<long>((n + 255) / 256, 4096));
  switch (C) {
    case 8:
    case 16:
    case 32: hipLaunchKernelGGL(k_head<1>, g, dim3(256), 0, s, src, C, wt, bias, relu, out, n); break;
    case 64: hipLaunchKernelGGL(k_head<2>, g, dim3(256), 0, s, src, C, wt, bias, relu, out, n); break;
    case 128: hipLaunchKernelGGL(k_head<4>, g, dim3(256), 0, s, src, C, wt, bias, relu, out, n); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int mse_blocks(long n) { return std::min(ew_grid((size_t)n), 512); }

hipError_t launch_mse(const float* y, const float* t, long n, float pos_w, uint16_t* g, float* part, hipStream_t s) {
  hipLaunchKernelGGL(k_mse, dim3(mse_blocks(n)), dim3(256), 0, s, y, t, n, 1.f / (float)n, pos_w, g, part);
  return hipGetLastError();
}

hipError_t launch_pack(PackTable& tab, hipStream_t s) {
  int blocks = 0;
  for (int k = 0; k < tab.n; ++k) {
    tab.e[k].block0 = blocks;
    blocks += (tab.e[k].T * tab.e[k].Npad * tab.e[k].Cpad + 255) / 256;
  }
  hipLaunchKernelGGL(k_pack, dim3(blocks), dim3(256), 0, s, tab);
  return hipGetLastError();
}

}  // namespace rihvr
