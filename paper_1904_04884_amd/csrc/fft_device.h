// Device-side FFT building blocks for gfx950: self-sorting (Stockham) radix
// 2/3/4/8/12 passes, complex helpers, and the compile-time radix plan.  A
// transform of length L is processed by T = L/P threads, each owning P points
// per pass (P divisible by every radix used).
//
// Stockham pass with radix R and span p (product of the radices already
// applied), for butterfly i in [0, L/R), k = i mod p:
//     u_r = a[i + r L/R] * w^(r k / (p R)),  r = 0..R-1,  w = exp(-+2 pi i)
//     U   = DFT_R(u)
//     b[(i - k) R + k + r p] = U_r
// After the last pass the data are in natural order.  With thread t taking the
// butterflies i = t + b T, the first pass's inputs and the last pass's outputs
// are the elements t + s T, s = 0..P-1, so a transform starts and ends in
// registers and only the exchanges between passes go through LDS.
#pragma once
#include <hip/hip_runtime.h>

namespace rihvr {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// multiply by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 mul_mi(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// ---------------------------------------------------------------------------
// Small DFTs, X_q = sum_m x_m exp(-+2 pi i m q / R)  (sign + for INV)
// ---------------------------------------------------------------------------
template <int R, bool INV> struct Dft;

template <bool INV> struct Dft<2, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <bool INV> struct Dft<3, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float c = -0.5f, s = 0.86602540378443864676f;  // cos, sin of 2 pi / 3
    float2 s12 = cadd(v[1], v[2]);
    float2 d12 = csub(v[1], v[2]);
    float2 m = make_float2(v[0].x + c * s12.x, v[0].y + c * s12.y);
    // forward: X1 = m - i s d, X2 = m + i s d
    float2 isd = INV ? make_float2(-s * d12.y, s * d12.x) : make_float2(s * d12.y, -s * d12.x);
    v[0] = cadd(v[0], s12);
    v[1] = cadd(m, isd);
    v[2] = csub(m, isd);
  }
};

template <bool INV> struct Dft<4, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    float2 t2 = cadd(v[1], v[3]), t3 = mul_mi<INV>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
  }
};

template <bool INV> struct Dft<8, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float h = 0.70710678118654752440f;
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    Dft<4, INV>::run(e);
    Dft<4, INV>::run(o);
    // twiddles exp(-+ i pi q / 4), q = 1..3
    float2 o1 = INV ? make_float2(h * (o[1].x - o[1].y), h * (o[1].x + o[1].y))
                    : make_float2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
    float2 o2 = mul_mi<INV>(o[2]);
    float2 o3 = INV ? make_float2(-h * (o[3].x + o[3].y), h * (o[3].x - o[3].y))
                    : make_float2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
  }
};

// 12 = 3 x 4 without twiddles (Good-Thomas): with input n = (4 n1 + 3 n2) mod 12
// and output q = (4 q1 + 9 q2) mod 12 the transform is a 3-point one over n1 and
// a 4-point one over n2.
template <bool INV> struct Dft<12, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 a[3][4];
#pragma unroll
    for (int n1 = 0; n1 < 3; ++n1) {
#pragma unroll
      for (int n2 = 0; n2 < 4; ++n2) a[n1][n2] = v[(4 * n1 + 3 * n2) % 12];
      Dft<4, INV>::run(a[n1]);
    }
#pragma unroll
    for (int q2 = 0; q2 < 4; ++q2) {
      float2 c[3] = {a[0][q2], a[1][q2], a[2][q2]};
      Dft<3, INV>::run(c);
#pragma unroll
      for (int q1 = 0; q1 < 3; ++q1) v[(4 * q1 + 9 * q2) % 12] = c[q1];
    }
  }
};

// ---------------------------------------------------------------------------
// Compile-time radix plan.  L = 2^a or 3 * 2^a.  A pass with the factor 3 comes
// first (radix 12 where P allows), then radix 8 while it divides both the
// remaining length and P, then 4 / 2.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int next_radix(int rem, int P) {
  return (rem % 12 == 0 && P % 12 == 0) ? 12
       : (rem % 3 == 0) ? 3
       : (rem % 8 == 0 && P % 8 == 0) ? 8
       : (rem % 4 == 0 && P % 4 == 0) ? 4
       : 2;
}

__host__ __device__ constexpr bool valid_len(int L) {
  int n = L;
  if (n % 3 == 0) n /= 3;
  while (n % 2 == 0) n /= 2;
  return n == 1;
}

// Points per thread for a transform of length L.
__host__ __device__ constexpr int points_per_thread(int L) {
  return (L % 3 == 0) ? (L >= 12 ? 12 : L) : (L >= 8 ? 8 : L);
}

// Ordering point between the LDS writes and reads of a transform: a block
// barrier, or, when each transform lies inside one wavefront (WAVE), only an
// ordering of that wave's LDS accesses (the LDS executes one wave's operations
// in issue order), so that waves holding different transforms never wait for
// each other.
template <bool WAVE>
__device__ __forceinline__ void lds_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// The first pass writes its R outputs side by side, so threads write R elements
// apart: on the same banks for even R.  That exchange therefore skips one element
// in every fft_pad (0: none).
__host__ __device__ constexpr int fft_pad(int L, int P) {
  const int R = next_radix(L, P);
  return R == L ? 0 : (R == 8 ? 8 : (R == 12 || R == 4 ? 4 : 0));
}
// Elements (times the stride S) of the LDS buffer of a transform.
__host__ __device__ constexpr int fft_buf_len(int L, int P) { return L + (fft_pad(L, P) > 0 ? L / fft_pad(L, P) : 0); }

// One pass and the ones after it.  v holds the elements t + s T on entry and
// on return.  An exchange waits before it writes (the one before may still be
// read) and before it reads; two buffers in turn, with one barrier per exchange,
// measured no faster in the column kernels at 1024 and 512 points.
template <int L, int P, int S, int TWS, int p, int rem, bool INV, bool WAVE>
__device__ __forceinline__ void fft_passes(float2 (&v)[P], float2* buf, int t, const float2* __restrict__ tw) {
  constexpr int R = next_radix(rem, P), T = L / P, NB = P / R;
  static_assert(P % R == 0, "radix must divide the points per thread");
  float2 u[NB][R];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int r = 0; r < R; ++r) u[b][r] = v[b + r * NB];
    if constexpr (p > 1) {
      const int k = (t + b * T) % p;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const float2 w = tw[(r * k * (L / (p * R))) * TWS];
        u[b][r] = INV ? cmulc(u[b][r], w) : cmul(u[b][r], w);
      }
    }
    Dft<R, INV>::run(u[b]);
  }
  if constexpr (rem == R) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < R; ++r) v[b + r * NB] = u[b][r];
  } else {
    constexpr int PAD = p == 1 ? fft_pad(L, P) : 0;
    auto at = [](int e) { return (PAD > 0 ? e + e / (PAD > 0 ? PAD : 1) : e) * S; };
    lds_sync<WAVE>();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = t + b * T, k = i % p, j = (i - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[at(j + r * p)] = u[b][r];
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int s = 0; s < P; ++s) v[s] = buf[at(t + s * T)];
    fft_passes<L, P, S, TWS, p * R, rem / R, INV, WAVE>(v, buf, t, tw);
  }
}

// Transform of length L (unscaled) of the elements t + s T in v, in place.
// Every thread of the block (of the wave, with WAVE) must call it.  Element e
// of an exchange sits at buf[e S] (plus padding); `tw` is a table
// exp(-2 pi i m / (L TWS)) read with stride TWS.
template <int L, int P, int S, int TWS, bool INV, bool WAVE>
__device__ __forceinline__ void fft_reg(float2 (&v)[P], float2* buf, int t, const float2* __restrict__ tw) {
  static_assert(valid_len(L), "length must be 2^a or 3*2^a");
  fft_passes<L, P, S, TWS, 1, L, INV, WAVE>(v, buf, t, tw);
}

}  // namespace rihvr
