// FP64 plans: the hologram model, its adjoint and the pieces of the FISTA
// iteration in double precision, for separating defects from FP32 rounding.
//
// The operator is the same angular-spectrum model (section "Methodology",
// Eq. 2 with the propagator A x = Re(sum_j IFFT2(FFT2(x_j) H_j))) from the
// same FP64 plan tables (theta, carriers), but computed plainly: complex
// transforms of whole planes (no packed half spectra), every plane's spectrum
// held at once, the filter cos(2 pi frac(z_j theta + c_j)) applied and summed
// over planes one frequency at a time.  The transforms are mixed-radix (4, 2, 3)
// Stockham FFTs of several lines per block, in LDS.  The FP32 path's kernels are
// specialised for FP32 register and LDS budgets; this path is a second
// implementation at 1e-9 of the FP64 oracle.
#include <hip/hip_runtime.h>

#include "rihvr_internal.h"

namespace rihvr {
namespace {

constexpr int kFThreads = 256;

__device__ __forceinline__ double2 cmul64(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// cos(2 pi frac(z_j theta(f) + c_j)) at grid frequency (ky, kx): theta is
// tabulated for kx in [0, nx/2] (it depends on fx^2 only).
__device__ __forceinline__ double filt64(const Plan64Tables& t, int j, int ky, int kx) {
  const int kk = kx <= t.m ? kx : t.nx - kx;
  const double th = t.theta[(size_t)ky * (t.m + 1) + kk];
  const double2 zc = t.zc[j];
  double ph = fma(zc.x, th, zc.y);
  ph -= floor(ph);
  return cospi(2.0 * ph);
}

// Transforms of length N of `group` lines per block: rows (COL = false) or
// adjacent columns of a plane.  Forward: exp(-2 pi i k n / N); inverse:
// exp(+...), both unscaled.  tw[k] = exp(-2 pi i k / N).
// Input: the complex data, a real volume, or (columns) the spectrum of one plane
// times every plane's filter.  Output: the complex data in place, or the real
// part as out = ca * value + cb * base.
//
// Bound by LDS exchanges and, at small volumes, by the latency of few blocks:
// radix 4 halves the stages of radix 2, several lines a block make 128-byte
// column segments of 16-byte ones and the conversions' and the filter's passes
// ride on the loads and stores (192 x 128 x 24, forward and adjoint of an
// iteration: 300 us with a line per block, now 74).
enum { IN64_COMPLEX, IN64_REAL, IN64_SPREAD };
struct Fft64Args {
  double2* data;          // [planes][ny][nx]
  const double* real;     // IN64_REAL
  const double2* spec;    // IN64_SPREAD: [ny][nx]
  double* out;            // real output (nullptr: complex in place)
  const double* base;     // nullable
  double ca, cb;
  const double2* tw;
  int N, group, inverse;
  Plan64Tables t;
};

template <bool COL, int IN>
__global__ void __launch_bounds__(kFThreads) k64_fft(Fft64Args f) {
  extern __shared__ double2 sh[];
  const int N = f.N, G = f.group, tl = kFThreads / G;   // tl threads per line (powers of two)
  const int g = COL ? (int)threadIdx.x % G : (int)threadIdx.x / tl, j0 = COL ? (int)threadIdx.x / G : (int)threadIdx.x % tl;
  const size_t np = (size_t)f.t.nx * f.t.ny;
  const int per = f.t.nx / G;   // column blocks of a plane
  const int plane = COL ? (int)blockIdx.x / per : 0, col = COL ? (int)(blockIdx.x % per) * G + g : 0;
  const size_t line = COL ? (size_t)plane * np + col : ((size_t)blockIdx.x * G + g) * (size_t)N;
  const size_t es = COL ? (size_t)f.t.nx : 1;
  auto at = [&](int k) { return COL ? k * G + g : g * N + k; };
  double2* a = sh;
  double2* b = sh + (size_t)N * G;
  for (int k = j0; k < N; k += tl) {
    const size_t i = line + (size_t)k * es;
    double2 v;
    if constexpr (IN == IN64_REAL) {
      v = make_double2(f.real[i], 0.0);
    } else if constexpr (IN == IN64_SPREAD) {
      const double2 r = f.spec[(size_t)k * f.t.nx + col];
      const double c = filt64(f.t, plane, k, col);
      v = make_double2(c * r.x, c * r.y);
    } else {
      v = f.data[i];
    }
    a[at(k)] = v;
  }
  __syncthreads();
  const double sg = f.inverse ? 1.0 : -1.0;
  int lg = 0, rem = N;   // ns = 2^lg points transformed so far (radix 3 comes last)
  while (rem > 1) {
    const int R = (rem & 3) == 0 ? 4 : ((rem & 1) == 0 ? 2 : 3);
    rem /= R;
    const int ns = 1 << lg, q = N / R;   // ts = rem: the twiddles' stride, N / (ns R)
    for (int j = j0; j < q; j += tl) {
      const int jm = j & (ns - 1), idx = ((j >> lg) << lg) * R + jm, w0 = jm * rem;
      auto in = [&](int r) {
        const double2 v = a[at(j + r * q)];
        if (lg == 0) return v;
        double2 w = f.tw[r * w0];
        if (f.inverse) w.y = -w.y;
        return cmul64(v, w);
      };
      const double2 v0 = a[at(j)], v1 = in(1);
      if (R == 4) {
        const double2 v2 = in(2), v3 = in(3);
        const double2 t0 = make_double2(v0.x + v2.x, v0.y + v2.y), t1 = make_double2(v0.x - v2.x, v0.y - v2.y);
        const double2 t2 = make_double2(v1.x + v3.x, v1.y + v3.y);
        // sg i (v1 - v3)
        const double2 t3 = make_double2(-sg * (v1.y - v3.y), sg * (v1.x - v3.x));
        b[at(idx)] = make_double2(t0.x + t2.x, t0.y + t2.y);
        b[at(idx + ns)] = make_double2(t1.x + t3.x, t1.y + t3.y);
        b[at(idx + 2 * ns)] = make_double2(t0.x - t2.x, t0.y - t2.y);
        b[at(idx + 3 * ns)] = make_double2(t1.x - t3.x, t1.y - t3.y);
      } else if (R == 2) {
        b[at(idx)] = make_double2(v0.x + v1.x, v0.y + v1.y);
        b[at(idx + ns)] = make_double2(v0.x - v1.x, v0.y - v1.y);
      } else {
        const double2 v2 = in(2);
        // exp(sg 2 pi i / 3) = -1/2 + sg i sqrt(3)/2
        const double h = 0.86602540378443864676 * sg;
        const double2 s = make_double2(v1.x + v2.x, v1.y + v2.y), d = make_double2(v1.x - v2.x, v1.y - v2.y);
        const double2 m = make_double2(v0.x - 0.5 * s.x, v0.y - 0.5 * s.y);
        b[at(idx)] = make_double2(v0.x + s.x, v0.y + s.y);
        b[at(idx + ns)] = make_double2(m.x - h * d.y, m.y + h * d.x);   // +- i h d
        b[at(idx + 2 * ns)] = make_double2(m.x + h * d.y, m.y - h * d.x);
      }
    }
    __syncthreads();
    double2* t = a;
    a = b;
    b = t;
    lg += R == 4 ? 2 : 1;
  }
  for (int k = j0; k < N; k += tl) {
    const size_t i = line + (size_t)k * es;
    const double2 v = a[at(k)];
    if (f.out == nullptr) f.data[i] = v;
    else f.out[i] = f.base != nullptr ? fma(f.ca, v.x, f.cb * f.base[i]) : f.ca * v.x;
  }
}

// S = sum_j X_j cos(phase_j).  A block takes 64 frequencies, a quarter of the
// planes per wavefront: the volume's planes alone fill few blocks.
__global__ void __launch_bounds__(kFThreads) k64_filter_sum(Plan64Tables t, const double2* __restrict__ X,
                                                            double2* __restrict__ S) {
  constexpr int W = kFThreads / 64;
  __shared__ double2 part[W][64];
  const size_t np = (size_t)t.nx * t.ny;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const size_t i = (size_t)blockIdx.x * 64 + lane;
  double2 acc = make_double2(0.0, 0.0);
  if (i < np) {
    const int ky = (int)(i / t.nx), kx = (int)(i % t.nx);
    for (int j = wv; j < t.nzp; j += W) {
      const double c = filt64(t, j, ky, kx);
      const double2 v = X[(size_t)j * np + i];
      acc.x = fma(c, v.x, acc.x);
      acc.y = fma(c, v.y, acc.y);
    }
  }
  part[wv][lane] = acc;
  __syncthreads();
  if (wv != 0 || i >= np) return;
  for (int w = 1; w < W; ++w) {
    acc.x += part[w][lane].x;
    acc.y += part[w][lane].y;
  }
  S[i] = acc;
}

__global__ void k64_fill(double* out, double v, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) out[i] = v;
}

// out = a x + b y (element by element; out may alias x or y)
__global__ void k64_axpby(double* out, double a, const double* x, double b, const double* y, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    out[i] = fma(a, x[i], b * y[i]);
}

// A wavefront per row: flags[row] = the row holds a value other than 0
__global__ void __launch_bounds__(kFThreads) k64_rowflags(const double* __restrict__ x, int nx, int nrow,
                                                          uint8_t* __restrict__ flags) {
  const int row = blockIdx.x * (kFThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= nrow) return;
  bool any = false;
  for (int i = lane; i < nx; i += 64) any |= x[(size_t)row * nx + i] != 0.0;
  const bool r = __ballot(any) != 0;
  if (lane == 0) flags[row] = r ? 1 : 0;
}

// per-block partial sums of (x - y)^2 over n elements, into part[blockIdx.x]
__global__ void __launch_bounds__(kFThreads) k64_sqdist(const double* x, const double* y, size_t n, double* part) {
  __shared__ double red[kFThreads / 64];
  double acc = 0.0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double d = x[i] - y[i];
    acc = fma(d, d, acc);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kFThreads / 64; ++w) s += red[w];
    part[blockIdx.x] = s;
  }
}

int fgrid(size_t n) {
  const size_t b = (n + kFThreads - 1) / kFThreads;
  return (int)(b > 8192 ? 8192 : (b == 0 ? 1 : b));
}

// Lines per block: up to 8 columns (128 bytes) or rows, whose two LDS buffers
// fit 64 KB, fewer where that leaves less than a block per compute unit or two.
int fft_group(int N, int lines) {
  int G = 8;
  while (G > 1 && (2 * (size_t)N * G * sizeof(double2) > 65536 || (G > 2 && lines / G < 256))) G /= 2;
  return G;
}
template <bool COL, int IN>
void launch_fft(Fft64Args f, int planes, hipStream_t s) {
  f.N = COL ? f.t.ny : f.t.nx;
  f.tw = COL ? f.t.tw_y : f.t.tw_x;
  const int lines = (COL ? f.t.nx : f.t.ny) * planes;
  f.group = fft_group(f.N, lines);   // divides lines: nx and ny are multiples of 8
  hipLaunchKernelGGL((k64_fft<COL, IN>), dim3(lines / f.group), dim3(kFThreads),
                     2 * (size_t)f.N * f.group * sizeof(double2), s, f);
}

}  // namespace

size_t f64_spectra_bytes(const Plan64Tables& t) {
  return (size_t)t.nx * t.ny * t.nzp * sizeof(double2);
}

hipError_t forward64(const Plan64Tables& t, const double* x, double* out, double2* X, double2* S, double cb,
                     const double* base, hipStream_t s) {
  const size_t np = (size_t)t.nx * t.ny;
  Fft64Args f{};
  f.t = t;
  f.data = X;
  f.real = x;
  launch_fft<false, IN64_REAL>(f, t.nzp, s);
  launch_fft<true, IN64_COMPLEX>(f, t.nzp, s);
  hipLaunchKernelGGL(k64_filter_sum, dim3((unsigned)((np + 63) / 64)), dim3(kFThreads), 0, s, t, X, S);
  f.data = S;
  f.inverse = 1;
  launch_fft<true, IN64_COMPLEX>(f, 1, s);
  f.out = out;
  f.base = base;
  f.ca = 1.0 / (double)np;
  f.cb = cb;
  launch_fft<false, IN64_COMPLEX>(f, 1, s);
  return hipGetLastError();
}

hipError_t adjoint64(const Plan64Tables& t, const double* y, double* out, double2* X, double2* S, double ca, double cb,
                     const double* base, hipStream_t s) {
  const size_t np = (size_t)t.nx * t.ny;
  Fft64Args f{};
  f.t = t;
  f.data = S;
  f.real = y;
  launch_fft<false, IN64_REAL>(f, 1, s);
  launch_fft<true, IN64_COMPLEX>(f, 1, s);
  f.data = X;
  f.spec = S;
  f.inverse = 1;
  launch_fft<true, IN64_SPREAD>(f, t.nzp, s);
  f.out = out;
  f.base = base;
  f.ca = ca / (double)np;
  f.cb = cb;
  launch_fft<false, IN64_COMPLEX>(f, t.nzp, s);
  return hipGetLastError();
}

hipError_t axpby64(double* out, double a, const double* x, double b, const double* y, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k64_axpby, dim3(fgrid(n)), dim3(kFThreads), 0, s, out, a, x, b, y, n);
  return hipGetLastError();
}

hipError_t rowflags64(const double* x, int nx, int nrow, uint8_t* flags, hipStream_t s) {
  hipLaunchKernelGGL(k64_rowflags, dim3((nrow + kFThreads / 64 - 1) / (kFThreads / 64)), dim3(kFThreads), 0, s, x, nx,
                     nrow, flags);
  return hipGetLastError();
}

hipError_t fill64(double* out, double v, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k64_fill, dim3(fgrid(n)), dim3(kFThreads), 0, s, out, v, n);
  return hipGetLastError();
}

hipError_t sqdist64(const double* x, const double* y, size_t n, double* part, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(k64_sqdist, dim3(nblocks), dim3(kFThreads), 0, s, x, y, n, part);
  return hipGetLastError();
}

}  // namespace rihvr
