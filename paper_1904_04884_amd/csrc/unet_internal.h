// Internal declarations of the warm-start U-Net kernels (unet.hip) used by the
// network driver (unet.cpp).  Not part of the public interface.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rihvr {

// Layer modes (see unet.hip); the 3x3x3 ones run k_conv3, the others the gather GEMM.
enum GatherMode {
  GG_CONV3_FWD = 0,  // rows: voxels; tap t reads voxel r + offset(t) (zero outside)
  GG_CONV3_BWD = 1,  // rows: voxels; tap t reads voxel r - offset(t)
  GG_UP_FWD = 2,     // rows: coarse voxels; column d*Cout + co is fine voxel 2q + d
  GG_UP_BWD = 3,     // rows: coarse voxels; tap d reads fine voxel 2q + d
  GG_POINT = 4,      // rows: voxels; one tap, same voxel (1x1x1 convolution)
};

// Input gradients of the up-convolution and the head (GG_UP_BWD, GG_POINT).
struct GatherGemmArgs {
  int mode;
  int D, H, W;             // grid of the rows (coarse grid for GG_UP_BWD)
  const uint16_t* src;     // BF16 channels-last source
  int src_cs;              // its channel stride
  int T, C;                // taps, channels per tap (multiple of 8)
  const uint16_t* wt;      // packed BF16 B[t][Npad][C]
  int N, Npad;             // real and padded (multiple of 16) output columns
  const uint16_t* mask;    // nullable: outputs where mask <= 0 become 0
  uint16_t* dst;           // BF16 [rows][N]
};
hipError_t launch_gather_gemm(const GatherGemmArgs& a, hipStream_t s);

struct UpArgs {
  int D, H, W;             // coarse grid
  const uint16_t* src;     // [voxels][cu]
  int cu, c;               // input and output channels
  const uint16_t* wt;      // packed BF16 [8 c][cu]
  const float* bias;
  uint16_t* dst;           // [fine voxels][c]
};
hipError_t launch_up_fwd(const UpArgs& a, hipStream_t s);
hipError_t launch_head(const uint16_t* src, int C, const uint16_t* wt, const float* bias, int relu, float* out, long n,
                       hipStream_t s);

// 3x3x3 layer (forward, or its input gradient with the per-tap transposed weights).
struct ConvArgs {
  int bwd;
  int D, H, W;
  const uint16_t* src;     // channels [0, C/2) of the input (all of them when C = 8), stride src_cs
  const uint16_t* src2;    // channels [C/2, C)
  int src_cs;
  const float* src32;      // instead of src, C = 8: channel 0 is scale * src32 rounded to BF16, the others 0
  float scale;
  int C;                   // input channels: 8, 16, 32, 64 or 128
  const uint16_t* wt;      // packed BF16 B[27][Npad][C]
  int N, Npad;             // real (multiple of 8) and padded output channels
  const float* bias;       // nullable
  int relu;
  const uint16_t* mask;    // nullable: outputs where mask <= 0 become 0 (same voxel and channel)
  int mask_cs;
  uint16_t* dst;           // channels [0, nsplit)
  uint16_t* dst2;          // channels [nsplit, N)
  int nsplit, dst_cs;
  int zrun;                // set by the launcher
};
hipError_t launch_conv3(ConvArgs a, hipStream_t s);

// Weight and bias gradient of one layer: per-block partials, added in order
// (with the loss and, for lr > 0, the Adam update) by launch_finish_grads, so
// a training step gives the same bits on every run.
struct WgradArgs {
  int mode;                // GG_CONV3_FWD, GG_UP_FWD (coarse rows) or GG_POINT
  int D, H, W;             // row grid
  const uint16_t* g;       // gradient w.r.t. the layer output (masked)
  int g_cs, N;
  const uint16_t* s;       // layer input, channels [0, ssplit)
  const uint16_t* s2;      // channels [ssplit, C): channel c at s2 + c
  int ssplit, s_cs, C;
  const float* s32;        // instead of s, C = 1: scale * s32 rounded to BF16
  float scale;
  float* part;             // [blocks][t][C][N]
  float* bpart;            // [blocks (x 8 up-convolution taps)][N]
  int Cpad, taps;          // set by launch_wgrad
};
int wgrad_blocks(int mode, int D, int H, int W, int N, int C);
hipError_t launch_wgrad(WgradArgs a, int blocks, hipStream_t s);

struct GradEntry {
  const float* part;       // [parts][count]
  float* out;
  long param;              // first parameter of the entry, or -1 (the loss)
  int count, parts;
  int block0;              // set by launch_finish_grads
};
struct GradTable {
  int n;
  GradEntry e[2 * 28 + 1]; // weights and biases of at most 28 layers, the loss
};
struct AdamArgs {
  float *w, *m, *v;
  float lr, b1, b2, a1, a2, eps, c1, c2;
};
hipError_t launch_finish_grads(GradTable& tab, const AdamArgs& ad, hipStream_t s);

hipError_t launch_pool_fwd(const uint16_t* x, uint16_t* y, uint8_t* idx, int C, int D, int H, int W, hipStream_t s);
hipError_t launch_pool_bwd(const uint16_t* gy, const uint8_t* idx, const uint16_t* y, uint16_t* g, int C, int D, int H,
                           int W, hipStream_t s);   // D, H, W: coarse dims
int mse_blocks(long n);
// g: [n][8]; part: mse_blocks(n) floats
hipError_t launch_mse(const float* y, const float* t, long n, float pos_w, uint16_t* g, float* part, hipStream_t s);

struct PackEntry {
  const float* w;
  uint16_t* out;
  int T, cin, cout, kind, Npad, Cpad;
  int block0;              // set by launch_pack
};
struct PackTable {
  int n;
  PackEntry e[2 * 28];     // forward and input-gradient weights of at most 28 layers
};
hipError_t launch_pack(PackTable& tab, hipStream_t s);

}  // namespace rihvr
