// Particle tracking back end on gfx950: segmentation of a reconstructed volume
// into objects and their weighted centroids (section "Methodology", the
// segmentation paragraph: a threshold at a small fraction of the maximum and a
// minimum object volume), linking of the objects of successive frames by the
// method of Crocker & Grier and track bookkeeping (section "Synthetic
// Turbulent Flow": weighted centroids, maximum displacement per frame,
// minimum track duration).
//
// Segmentation.  Voxels above rel * max(x) are foreground.  The volume is read
// twice, for its maximum and for a bit mask of the foreground (a wavefront's
// ballot is a 64-voxel word of a row); everything after that works on the mask,
// 1/32 of the volume, and on the runs of set bits in its words.  Connected
// components (26-connectivity) by union-find over the runs: a run starts as its
// own root and unites with the runs it touches in the word before it and in the
// four neighbour rows of smaller index, always linking the larger root below
// the smaller with an atomic minimum, so the root of a component ends as its
// first run in raster order, which starts at the component's smallest linear
// index.  Two runs of a row never start at x = 2k and 2k + 1 (words begin at
// even x), so a run's label sits at half its start: ceil(nx / 2) labels a row.
// Roots are then numbered in order (counts per block, each block adding those
// before it, ranking); a root's label takes its number with the top bit set.
// Voxel counts and FP64 sums of x and x times each coordinate are formed per
// run and added to the object's with atomics; objects with at least min_voxels
// voxels are written in number order with their weighted centroid.
//
// 512^2 x 128, 1500 particles: the seven launches take 165 us, of which the
// two reads of the volume (134 MB, 28 us each at the copy rate) 84; a label
// word per voxel with every voxel visited in each of eight passes took 650.
//
// Linking.  For two frames of object positions, the candidate links are the
// pairs within the maximum displacement (physical units through a per-axis
// spacing).  Sources that share candidate targets form subnetworks (union-find
// over sources and targets); the assignments of a subnetwork are enumerated --
// sources in ascending order, each taking one of its candidates by increasing
// distance or none, none last -- and the first one of least sum(d^2) +
// max_disp^2 * (unlinked sources) is kept.  Distances and sums are formed with
// rounded FP64 operations in a fixed order, so equal costs resolve the same way
// on every run.  A wavefront takes a source (its lanes the targets) and a
// subnetwork (its lanes the sources it may hold): with a thread each, 1500
// objects left the device to a few wavefronts' serial scans (candidates 373 us,
// search 374 us; now 12 and 11).
#include <hip/hip_runtime.h>

#include <cstdio>

#include "../../include/rihvr.h"

namespace rihvr {
ri_status set_error(ri_status st, const char* msg);
}

namespace {

constexpr uint32_t kRootMark = 0x80000000u;  // a numbered root's label
constexpr int kDetThreads = 256;
constexpr int kDetBlocks = 2048;             // most blocks of the numbering passes
constexpr int kDetMaxBlocks = 1024;          // most blocks of the maximum
constexpr int kDetWords = 8;                 // words a wavefront masks at a time (loads in flight)
constexpr uint32_t kDetSplitWords = 1u << 16;   // up to here a word's runs go to eight threads
constexpr int kDetManyRuns = 8;              // from here on they go to a wavefront
constexpr int kLinkMaxCand = 8;              // candidates kept per source
constexpr int kLinkMaxSubnet = 8;            // sources per subnetwork
constexpr int kLinkOver = 0x100;             // on a count of candidates: there were more

__device__ __forceinline__ uint32_t find_root(const uint32_t* lab, uint32_t i) {
  uint32_t p = lab[i];
  while (p != i) {
    i = p;
    p = lab[i];
  }
  return i;
}

// Link the components of a and b: the larger root is set below the smaller by
// an atomic minimum; when another thread relinked it first, retry from there.
__device__ __forceinline__ void unite(uint32_t* lab, uint32_t a, uint32_t b) {
  while (true) {
    a = find_root(lab, a);
    b = find_root(lab, b);
    if (a == b) return;
    if (a > b) {
      const uint32_t t = a;
      a = b;
      b = t;
    }
    const uint32_t old = atomicMin(&lab[b], a);
    if (old == b) return;
    b = old;
  }
}

// Clearing by a kernel rather than a memset, so that a caller may capture the
// sequence into a HIP graph.
__global__ void k_fill_u32(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Foreground mask geometry: words of 64 voxels, wpr per row; labels hx per row.
struct MaskGeom {
  int nx, ny, nz;
  uint32_t wpr, hx, words;
};
__device__ __forceinline__ uint32_t label_of(const MaskGeom& g, uint32_t row, uint32_t x) { return row * g.hx + (x >> 1); }
// First bit of the run of m that holds bit b, and the bits of that run.
__device__ __forceinline__ int run_start(uint64_t m, int b) {
  const uint64_t t = ~m & ((1ull << b) - 1ull);
  return t ? 64 - __clzll((long long)t) : 0;
}
__device__ __forceinline__ uint64_t run_bits(uint64_t m, int start) {
  const uint64_t t = ~(m >> start);            // its lowest set bit ends the run
  const int len = t ? __ffsll((unsigned long long)t) - 1 : 64;
  return (len >= 64 ? ~0ull : (1ull << len) - 1ull) << start;
}

__device__ __forceinline__ float block_max(float m, float* red) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  for (int w = 0; w < kDetThreads / 64; ++w) m = fmaxf(m, red[w]);
  return m;
}

// Largest value (at least 0) of each block's share of x; clears the object sums.
// Bound by the read of x; 16-byte loads from its first aligned element on.
__global__ void __launch_bounds__(kDetThreads) k_det_max(const float* __restrict__ x, size_t n, float* __restrict__ part,
                                                         uint32_t* __restrict__ cnt, double* __restrict__ sums,
                                                         size_t max_comp) {
  __shared__ float red[kDetThreads / 64];
  const size_t tid = (size_t)blockIdx.x * kDetThreads + threadIdx.x, nt = (size_t)gridDim.x * kDetThreads;
  for (size_t i = tid; i < max_comp; i += nt) cnt[i] = 0;
  for (size_t i = tid; i < 4 * max_comp; i += nt) sums[i] = 0.0;
  float m = 0.f;
  const size_t mis = ((uintptr_t)x >> 2) & 3;
  const size_t head = mis ? (n < 4 - mis ? n : 4 - mis) : 0;
  const size_t n4 = (n - head) / 4;
  const float4* x4 = reinterpret_cast<const float4*>(x + head);
  size_t i = tid;
  for (; i + 3 * nt < n4; i += 4 * nt) {
    float4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = x4[i + k * nt];
#pragma unroll
    for (int k = 0; k < 4; ++k) m = fmaxf(m, fmaxf(fmaxf(v[k].x, v[k].y), fmaxf(v[k].z, v[k].w)));
  }
  for (; i < n4; i += nt) {
    const float4 v = x4[i];
    m = fmaxf(m, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
  }
  if (tid < head) m = fmaxf(m, x[tid]);
  if (tid < n - head - 4 * n4) m = fmaxf(m, x[head + 4 * n4 + tid]);
  m = block_max(m, red);
  if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// Foreground mask, and every run's label its own.  Bound by the read of x.
__global__ void __launch_bounds__(kDetThreads) k_det_mask(const float* __restrict__ x, MaskGeom g,
                                                          const float* __restrict__ part, int nparts, double rel,
                                                          uint64_t* __restrict__ mask, uint32_t* __restrict__ lab) {
  __shared__ float red[kDetThreads / 64];
  float m = 0.f;
  for (int i = threadIdx.x; i < nparts; i += kDetThreads) m = fmaxf(m, part[i]);
  m = block_max(m, red);
  const double thr = rel * (double)m;
  const bool any = m > 0.f;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t nw = gridDim.x * (kDetThreads / 64);
  for (uint64_t w0 = (uint64_t)__builtin_amdgcn_readfirstlane(blockIdx.x * (kDetThreads / 64) + (threadIdx.x >> 6)) * kDetWords;
       w0 < g.words; w0 += (uint64_t)nw * kDetWords) {
    float v[kDetWords];
    uint32_t row[kDetWords], xx[kDetWords];
    uint32_t r = (uint32_t)w0 / g.wpr, wx = (uint32_t)w0 % g.wpr;
#pragma unroll
    for (int k = 0; k < kDetWords; ++k) {
      row[k] = r;
      xx[k] = wx * 64 + lane;
      v[k] = (w0 + k < g.words && xx[k] < (uint32_t)g.nx) ? x[(size_t)r * g.nx + xx[k]] : -1.f;
      if (++wx == g.wpr) {
        wx = 0;
        ++r;
      }
    }
    uint64_t mine = 0;
#pragma unroll
    for (int k = 0; k < kDetWords; ++k) {
      const bool in = w0 + k < g.words && xx[k] < (uint32_t)g.nx;
      const uint64_t b = __ballot(in && any && (double)v[k] > thr);
      if (lane == (uint32_t)k) mine = b;
      if (((b & ~(b << 1)) >> lane) & 1ull) {
        const uint32_t l = label_of(g, row[k], xx[k]);
        lab[l] = l;
      }
    }
    if (lane < kDetWords && w0 + lane < g.words) mask[w0 + lane] = mine;
  }
}

// Unites the run of row `row` that starts at bit st of word m (word wx of the row) with
// those it touches in a neighbour row of smaller index, k = (z, y - 1), then
// (z - 1, y - 1 .. y + 1); k = 0 also with the word before.
__device__ __forceinline__ void unite_run(const uint64_t* mask, const MaskGeom& g, uint32_t* lab, uint32_t row, uint32_t wx,
                                          uint64_t m, int st, int k) {
  const int dy = k == 0 ? -1 : k - 2, dz = k == 0 ? 0 : -1;
  const int y = (int)(row % g.ny), z = (int)(row / g.ny);
  const uint64_t run = run_bits(m, st);
  const uint32_t l = label_of(g, row, wx * 64 + st);
  const bool left = wx > 0 && (run & 1ull), right = wx + 1 < g.wpr && (run >> 63);
  if (k == 0 && left) {
    const uint64_t a = mask[(size_t)row * g.wpr + wx - 1];
    if (a >> 63) unite(lab, l, label_of(g, row, (wx - 1) * 64 + run_start(a, 63)));
  }
  if (z + dz < 0 || y + dy < 0 || y + dy >= g.ny) return;
  const uint32_t nr = (uint32_t)((int64_t)row + (int64_t)dz * g.ny + dy);
  const uint64_t* nb = mask + (size_t)nr * g.wpr + wx;
  const uint64_t c = nb[0];
  for (uint64_t h = (run | (run << 1) | (run >> 1)) & c; h != 0;) {
    const int s = run_start(c, __ffsll((unsigned long long)h) - 1);
    h &= ~run_bits(c, s);
    unite(lab, l, label_of(g, nr, wx * 64 + s));
  }
  if (left) {
    const uint64_t a = nb[-1];
    if (a >> 63) unite(lab, l, label_of(g, nr, (wx - 1) * 64 + run_start(a, 63)));
  }
  if (right && (nb[1] & 1ull)) unite(lab, l, label_of(g, nr, (wx + 1) * 64));
}

// Unites every run with those it touches in the word before and in the four neighbour
// rows of smaller index.  Bound by chains of dependent loads, so a word's rows go to four
// threads, and where that leaves the device part empty (kDetSplitWords) the runs that
// start in its eighths to 2^ps = 8; most words are empty.  A word of many runs is taken
// by the whole wavefront, a lane for each: neighbouring labels in one load.  512^2 x 128
// with every other column set: 2.85 ms with four threads a word, 0.8 now; 64^2 x 40:
// 255 us, 35 now.
__global__ void __launch_bounds__(kDetThreads) k_det_union(const uint64_t* __restrict__ mask, MaskGeom g, int ps,
                                                           uint32_t* lab) {
  const int lane = threadIdx.x & 63, k = threadIdx.x & 3;
  const int part = (threadIdx.x >> 2) & ((1 << ps) - 1), bits = 64 >> ps;
  const uint64_t mine = (~0ull >> (64 - bits)) << (part * bits);   // where this thread's runs start
  const uint32_t per = kDetThreads >> (2 + ps);
  for (uint64_t i0 = (uint64_t)blockIdx.x * per; i0 < g.words; i0 += (uint64_t)gridDim.x * per) {
    const uint64_t i = i0 + (threadIdx.x >> (2 + ps));
    const uint64_t m = i < g.words ? mask[i] : 0ull, starts = m & ~(m << 1);
    const bool many = __popcll(starts) > kDetManyRuns;
    if (!many) {
      const uint32_t row = (uint32_t)i / g.wpr, wx = (uint32_t)i % g.wpr;
      for (uint64_t q = starts & mine; q != 0; q &= q - 1)
        unite_run(mask, g, lab, row, wx, m, __ffsll((unsigned long long)q) - 1, k);
    }
    for (uint64_t h = __ballot(many && part == 0 && k == 0); h != 0; h &= h - 1) {
      const uint32_t w = (uint32_t)__shfl((int)(uint32_t)i, __ffsll((unsigned long long)h) - 1, 64);
      const uint64_t mw = mask[w];
      if (((mw & ~(mw << 1)) >> lane) & 1ull)
        for (int kk = 0; kk < 4; ++kk) unite_run(mask, g, lab, w / g.wpr, w % g.wpr, mw, lane, kk);
    }
  }
}

// f(x, label, whether it is a root) for the runs of word i in order, four label loads in
// flight.
template <class F>
__device__ __forceinline__ void for_runs(const uint64_t m, const MaskGeom& g, const uint32_t* lab, uint64_t i, F f) {
  const uint32_t row = (uint32_t)i / g.wpr, wx = (uint32_t)i % g.wpr;
  for (uint64_t q = m & ~(m << 1); q != 0;) {
    uint32_t x[4], l[4];
    bool on[4], root[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      on[k] = q != 0;
      x[k] = wx * 64 + (on[k] ? __ffsll((unsigned long long)q) - 1 : 0);
      l[k] = label_of(g, row, x[k]);
      q &= q - 1;   // (0 stays 0)
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) root[k] = on[k] && lab[l[k]] == l[k];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (on[k]) f(x[k], l[k], root[k]);
  }
}

// Roots among the runs of word i.
__device__ __forceinline__ uint32_t roots_of(const uint64_t* mask, const MaskGeom& g, const uint32_t* lab, uint64_t i) {
  uint32_t c = 0;
  for_runs(mask[i], g, lab, i, [&](uint32_t, uint32_t, bool root) { c += root ? 1u : 0u; });
  return c;
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t c, uint32_t* red) {
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  uint32_t t = 0;
  for (int w = 0; w < kDetThreads / 64; ++w) t += red[w];
  return t;
}

// Roots in each block's chunk of words.
__global__ void __launch_bounds__(kDetThreads) k_det_count_roots(const uint64_t* __restrict__ mask, MaskGeom g,
                                                                 const uint32_t* __restrict__ lab, uint32_t chunk,
                                                                 uint32_t* __restrict__ counts) {
  __shared__ uint32_t red[kDetThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * chunk;
  uint32_t c = 0;
  for (uint32_t k = threadIdx.x; k < chunk && base + k < g.words; k += kDetThreads) c += roots_of(mask, g, lab, base + k);
  c = block_sum_u32(c, red);
  if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

// Number the roots in raster order; a root's label becomes its number with the
// top bit set, and the linear index of its first voxel is recorded (numbers
// below max_comp).  The last block leaves the number of roots in *total.
__global__ void __launch_bounds__(kDetThreads) k_det_number(const uint64_t* __restrict__ mask, MaskGeom g, uint32_t* lab,
                                                            uint32_t chunk, const uint32_t* __restrict__ counts,
                                                            uint32_t max_comp, uint32_t* __restrict__ first,
                                                            uint32_t* __restrict__ total) {
  __shared__ uint32_t red[kDetThreads / 64], wsum[kDetThreads / 64];
  const uint64_t base = (uint64_t)blockIdx.x * chunk;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t before = 0;
  for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kDetThreads) before += counts[k];
  uint32_t run = block_sum_u32(before, red);
  for (uint32_t k = 0; k < chunk; k += kDetThreads) {
    const uint64_t i = base + k + threadIdx.x;
    const uint32_t c = i < g.words ? roots_of(mask, g, lab, i) : 0u;
    uint32_t incl = c;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t t = __shfl_up(incl, off, 64);
      incl += lane >= off ? t : 0u;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t id = run + incl - c, tot = 0;
    for (int w = 0; w < kDetThreads / 64; ++w) {
      id += w < wv ? wsum[w] : 0u;
      tot += wsum[w];
    }
    if (c != 0) {
      const uint32_t row = (uint32_t)i / g.wpr;
      for_runs(mask[i], g, lab, i, [&](uint32_t x, uint32_t l, bool root) {
        if (!root) return;
        lab[l] = kRootMark | id;
        if (id < max_comp) first[id] = (uint32_t)((size_t)row * g.nx + x);
        ++id;
      });
    }
    run += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *total = run;
}

// Sums of the objects.  A block adds its runs per object in LDS (a hash table, emptied
// into the objects' sums once at the end): where many runs of one object follow each
// other, global atomics on the same few words take turns.  512^2 x 128 with every other
// column of x set: 53 ms with five global atomics a run, 2.0 now; two frames of 1500
// particles segmented, linked and numbered: 402 -> 365 us.
// A thread takes the runs that start in a word (its eighths, as k_det_union).
constexpr int kDetSlots = 512, kDetProbes = 8;

__global__ void __launch_bounds__(kDetThreads) k_det_stats(const float* __restrict__ x, const uint64_t* __restrict__ mask,
                                                           MaskGeom g, int ps, const uint32_t* __restrict__ lab,
                                                           uint32_t max_comp, uint32_t* cnt,
                                                           double* sums /* [4][max_comp]: w, wz, wy, wx */) {
  __shared__ uint32_t s_id[kDetSlots], s_cnt[kDetSlots];
  __shared__ double s_sum[4][kDetSlots];
  const int part = threadIdx.x & ((1 << ps) - 1), bits = 64 >> ps;
  const uint64_t mine = (~0ull >> (64 - bits)) << (part * bits);
  bool clean = false;   // the table is set up by the first words with a run
  for (uint64_t i0 = (uint64_t)blockIdx.x * (kDetThreads >> ps); i0 < g.words; i0 += (uint64_t)gridDim.x * (kDetThreads >> ps)) {
    const uint64_t i = i0 + (threadIdx.x >> ps);
    const uint64_t m = i < g.words ? mask[i] : 0ull;
    if (!__syncthreads_or(m != 0)) continue;
    if (!clean) {
      clean = true;
      for (int e = threadIdx.x; e < kDetSlots; e += kDetThreads) {
        s_id[e] = ~0u;
        s_cnt[e] = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) s_sum[k][e] = 0.0;
      }
      __syncthreads();
    }
    const uint32_t row = (uint32_t)i / g.wpr, wx = (uint32_t)i % g.wpr;
    for (uint64_t q = m & ~(m << 1) & mine; q != 0; q &= q - 1) {
      const int st = __ffsll((unsigned long long)q) - 1;
      const int len = __popcll(run_bits(m, st));
      const uint32_t x0 = wx * 64 + st;
      uint32_t l = lab[label_of(g, row, x0)];
      while (!(l & kRootMark)) l = lab[l];
      const uint32_t id = l & ~kRootMark;
      if (id >= max_comp) continue;
      const float* src = x + (size_t)row * g.nx + x0;
      double sw = 0.0, sx = 0.0;
      for (int b0 = 0; b0 < len; b0 += 8) {   // eight loads in flight
        float v[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) v[b] = b0 + b < len ? src[b0 + b] : 0.f;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          sw += (double)v[b];
          sx += (double)v[b] * (double)(x0 + b0 + b);
        }
      }
      const double sz = sw * (double)(row / g.ny), sy = sw * (double)(row % g.ny);
      uint32_t h = (id * 2654435761u) >> 23;   // 9 bits: kDetSlots
      static_assert(kDetSlots == 512, "slots of the hash");
      bool held = false;
      for (int t = 0; t < kDetProbes && !held; ++t) {
        h = (h + (t > 0)) & (kDetSlots - 1);
        const uint32_t was = atomicCAS(&s_id[h], ~0u, id);
        held = was == ~0u || was == id;
      }
      if (held) {
        atomicAdd(&s_cnt[h], (uint32_t)len);
        unsafeAtomicAdd(&s_sum[0][h], sw);
        unsafeAtomicAdd(&s_sum[1][h], sz);
        unsafeAtomicAdd(&s_sum[2][h], sy);
        unsafeAtomicAdd(&s_sum[3][h], sx);
      } else {   // more objects than slots
        atomicAdd(&cnt[id], (uint32_t)len);
        unsafeAtomicAdd(&sums[id], sw);
        unsafeAtomicAdd(&sums[max_comp + id], sz);
        unsafeAtomicAdd(&sums[2 * (size_t)max_comp + id], sy);
        unsafeAtomicAdd(&sums[3 * (size_t)max_comp + id], sx);
      }
    }
  }
  if (!clean) return;
  __syncthreads();
  for (int e = threadIdx.x; e < kDetSlots; e += kDetThreads) {
    const uint32_t id = s_id[e];
    if (id == ~0u) continue;
    atomicAdd(&cnt[id], s_cnt[e]);
#pragma unroll
    for (int k = 0; k < 4; ++k) unsafeAtomicAdd(&sums[k * (size_t)max_comp + id], s_sum[k][e]);
  }
}

// Kept objects in number order (one block): out[k] = (z, y, x, w, count, first).
__global__ void k_det_finalize(const uint32_t* __restrict__ cnt, const double* __restrict__ sums,
                               const uint32_t* __restrict__ first, const uint32_t* ncomp_p, uint32_t max_comp,
                               int min_voxels, ri_object* out, int max_out, int32_t* counts) {
  __shared__ uint32_t wsum[kDetThreads / 64];
  const uint32_t ncomp = *ncomp_p;
  const uint32_t m = ncomp < max_comp ? ncomp : max_comp;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t run = 0;
  for (uint32_t base = 0; base < m; base += kDetThreads) {
    const uint32_t id = base + threadIdx.x;
    const bool keep = id < m && cnt[id] >= (uint32_t)min_voxels;
    const uint64_t mask = __ballot(keep);
    const uint32_t below = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wv] = (uint32_t)__popcll(mask);
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int w = 0; w < kDetThreads / 64; ++w) {
      before += w < wv ? wsum[w] : 0;
      tot += wsum[w];
    }
    if (keep) {
      const uint32_t k = run + before + below;
      if (k < (uint32_t)max_out) {
        const double w = sums[id];
        ri_object o;
        o.z = sums[max_comp + id] / w;
        o.y = sums[2 * (size_t)max_comp + id] / w;
        o.x = sums[3 * (size_t)max_comp + id] / w;
        o.weight = w;
        o.voxels = (double)cnt[id];
        o.first = (double)first[id];
        out[k] = o;
      }
    }
    run += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    counts[0] = (int32_t)run;
    counts[1] = (int32_t)ncomp;
  }
}

// ---------------------------------------------------------------------------
// Linking
// ---------------------------------------------------------------------------
struct LinkWs {
  int32_t* cand;      // [max_n0][kLinkMaxCand] target indices
  double* cand_d2;    // [max_n0][kLinkMaxCand]
  int32_t* ncand;     // [max_n0]
  uint32_t* parent;   // [max_n0 + max_n1] union-find over sources and targets
};

__device__ __forceinline__ double dist2(const ri_object& a, const ri_object& b, double sz, double sy, double sx) {
  // rounded FP64 products and sums in a fixed order (no contraction)
  const double dz = __dmul_rn(__dsub_rn(b.z, a.z), sz);
  const double dy = __dmul_rn(__dsub_rn(b.y, a.y), sy);
  const double dx = __dmul_rn(__dsub_rn(b.x, a.x), sx);
  return __dadd_rn(__dadd_rn(__dmul_rn(dz, dz), __dmul_rn(dy, dy)), __dmul_rn(dx, dx));
}

// Candidates of each source, sorted by (d2, j): a wavefront per source, its
// lanes taking 64 targets at a time; lane k holds candidate k.
__global__ void __launch_bounds__(kDetThreads)
k_link_candidates(const ri_object* __restrict__ prev, const int32_t* n0p, int max_n0, const ri_object* __restrict__ cur,
                  const int32_t* n1p, int max_n1, double sz, double sy, double sx, double r2, LinkWs w, int32_t* link,
                  int32_t* status) {
  const int n0 = min(*n0p, max_n0), n1 = min(*n1p, max_n1);
  if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;   // (set by the launches that follow)
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < max_n0 + max_n1; i += gridDim.x * blockDim.x)
    w.parent[i] = (uint32_t)i;
  const int lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * (kDetThreads / 64) + (threadIdx.x >> 6));
  if (i >= n0) return;
  if (lane == 0) link[i] = -1;
  const ri_object a = prev[i];
  int cj = -1, nc = 0, over = 0;
  double cd = 0.0;
  for (int j0 = 0; j0 < n1; j0 += 64) {
    const int j = j0 + lane;
    double d2 = 0.0;
    bool hit = false;
    if (j < n1) {
      d2 = dist2(a, cur[j], sz, sy, sx);
      hit = d2 <= r2;
    }
    // hits in ascending j, so equal distances keep index order
    for (uint64_t h = __ballot(hit); h != 0; h &= h - 1) {
      const int b = __ffsll((unsigned long long)h) - 1;
      const double db = __shfl(d2, b, 64);
      // candidates that stay ahead of it
      const int k = __popcll(__ballot(lane < nc && cd <= db));
      if (nc == kLinkMaxCand) {
        over = 1;
        if (k == kLinkMaxCand) continue;
      } else {
        ++nc;
      }
      const double cdp = __shfl_up(cd, 1, 64);
      const int cjp = __shfl_up(cj, 1, 64);
      if (lane == k) {
        cd = db;
        cj = j0 + b;
      } else if (lane > k) {
        cd = cdp;
        cj = cjp;
      }
    }
  }
  if (lane < nc) {
    w.cand[(size_t)i * kLinkMaxCand + lane] = cj;
    w.cand_d2[(size_t)i * kLinkMaxCand + lane] = cd;
  }
  if (lane == 0) w.ncand[i] = over ? nc | kLinkOver : nc;
}

__global__ void k_link_union(const int32_t* n0p, int max_n0, LinkWs w, int32_t* status) {
  const int n0 = min(*n0p, max_n0);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n0) return;
  int nc = w.ncand[i];
  if (nc & kLinkOver) {
    atomicOr(status, 2);
    nc &= ~kLinkOver;
    w.ncand[i] = nc;
  }
  for (int k = 0; k < nc; ++k) unite(w.parent, (uint32_t)i, (uint32_t)(max_n0 + w.cand[(size_t)i * kLinkMaxCand + k]));
}

// Every source's subnetwork root (its smallest source) in its parent word.
__global__ void k_link_roots(const int32_t* n0p, int max_n0, LinkWs w) {
  const int n0 = min(*n0p, max_n0);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n0) w.parent[i] = find_root(w.parent, (uint32_t)i);
}

// One wavefront per subnetwork: its lanes collect the members, lane 0 searches
// exhaustively in the fixed enumeration order.
__global__ void __launch_bounds__(kDetThreads)
k_link_solve(const int32_t* n0p, int max_n0, double r2, LinkWs w, int32_t* link, int32_t* status) {
  __shared__ int s_mem[kDetThreads / 64][kLinkMaxSubnet];
  __shared__ int s_nc[kDetThreads / 64][kLinkMaxSubnet];
  __shared__ int s_cand[kDetThreads / 64][kLinkMaxSubnet * kLinkMaxCand];
  __shared__ double s_d2[kDetThreads / 64][kLinkMaxSubnet * kLinkMaxCand];
  __shared__ int s_choice[kDetThreads / 64][kLinkMaxSubnet], s_best[kDetThreads / 64][kLinkMaxSubnet];
  __shared__ double s_cost[kDetThreads / 64][kLinkMaxSubnet + 1];
  const int n0 = min(*n0p, max_n0);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * (kDetThreads / 64) + wv);
  // (no barriers below: everything of a subnetwork stays in its wavefront)
  if (r >= n0 || w.ncand[r] == 0 || w.parent[r] != (uint32_t)r) return;
  auto settle = [] {   // a lane's LDS writes before the other lanes' reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int* mem = s_mem[wv];
  int nm = 0;
  for (int s0 = r; s0 < n0; s0 += 64) {   // members in ascending order
    const int s = s0 + lane;
    const bool in = s < n0 && w.parent[s] == (uint32_t)r && w.ncand[s] != 0;
    const uint64_t b = __ballot(in);
    const int k = nm + __popcll(b & ((1ull << lane) - 1ull));
    if (in && k < kLinkMaxSubnet) mem[k] = s;
    nm += __popcll(b);
    if (nm > kLinkMaxSubnet) {
      if (lane == 0) atomicOr(status, 1);
      return;
    }
  }
  settle();
  {
    const int q = lane / kLinkMaxCand, c = lane % kLinkMaxCand;
    static_assert(kLinkMaxSubnet * kLinkMaxCand == 64, "a lane per member and candidate");
    if (q < nm) {
      const int s = mem[q], nc = w.ncand[s];
      if (c == 0) s_nc[wv][q] = nc;
      s_cand[wv][lane] = c < nc ? w.cand[(size_t)s * kLinkMaxCand + c] : -1;
      s_d2[wv][lane] = c < nc ? w.cand_d2[(size_t)s * kLinkMaxCand + c] : r2;
    }
  }
  settle();
  if (lane != 0) return;
  // depth-first over (source k, choice c): c < ncand takes candidate c, c == ncand leaves it unlinked
  const int* cand = s_cand[wv];
  const double* d2 = s_d2[wv];
  const int* ncand = s_nc[wv];
  int *choice = s_choice[wv], *best = s_best[wv];
  double* cost = s_cost[wv];
  double best_cost = __builtin_huge_val();
  cost[0] = 0.0;
  int k = 0;
  choice[0] = -1;
  while (k >= 0) {
    const int nc = ncand[k];
    int c = choice[k] + 1;
    // next admissible choice: a candidate not taken by an earlier source, or "none"
    for (; c < nc; ++c) {
      const int j = cand[k * kLinkMaxCand + c];
      bool used = false;
      for (int q = 0; q < k; ++q)
        if (choice[q] < ncand[q] && cand[q * kLinkMaxCand + choice[q]] == j) used = true;
      if (!used) break;
    }
    if (c > nc) {   // every choice of this source tried: back up
      --k;
      continue;
    }
    choice[k] = c;
    const double add = c < nc ? d2[k * kLinkMaxCand + c] : r2;
    const double cst = __dadd_rn(cost[k], add);
    if (cst >= best_cost) continue;   // no strictly better assignment below this one
    if (k + 1 == nm) {
      best_cost = cst;
      for (int q = 0; q < nm; ++q) best[q] = choice[q];
      continue;
    }
    cost[k + 1] = cst;
    ++k;
    choice[k] = -1;
  }
  for (int q = 0; q < nm; ++q) link[mem[q]] = best[q] < ncand[q] ? cand[q * kLinkMaxCand + best[q]] : -1;
}

// Track ids of the current frame from the links of the previous one (one
// block): linked particles keep their source's id, the others open new ids in
// ascending particle order; track lengths grow by one for every id present.
__global__ void k_track_update(const int32_t* __restrict__ link, const int32_t* n0p, const int32_t* __restrict__ ids_prev,
                               const int32_t* n1p, int max_n1, int32_t* ids, int32_t* next_id, int32_t* track_len,
                               int max_tracks) {
  __shared__ uint32_t wsum[kDetThreads / 64];
  const int n1 = min(*n1p, max_n1), n0 = *n0p;
  for (int j = threadIdx.x; j < n1; j += kDetThreads) ids[j] = -1;
  __syncthreads();
  for (int i = threadIdx.x; i < n0; i += kDetThreads) {
    const int j = link[i];
    if (j >= 0 && j < n1) ids[j] = ids_prev[i];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int start = *next_id;
  uint32_t run = 0;
  for (int base = 0; base < n1; base += kDetThreads) {
    const int j = base + threadIdx.x;
    const bool fresh = j < n1 && ids[j] < 0;
    const uint64_t mask = __ballot(fresh);
    const uint32_t below = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wv] = (uint32_t)__popcll(mask);
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int w = 0; w < kDetThreads / 64; ++w) {
      before += w < wv ? wsum[w] : 0;
      tot += wsum[w];
    }
    if (fresh) ids[j] = start + (int)(run + before + below);
    run += tot;
    __syncthreads();
  }
  for (int j = threadIdx.x; j < n1; j += kDetThreads) {
    const int id = ids[j];
    if (id < max_tracks) atomicAdd(&track_len[id], 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) *next_id = start + (int)run;
}

__global__ void k_track_filter(const int32_t* __restrict__ track_len, const int32_t* n_tracks_p, int max_tracks,
                               int min_len, uint8_t* kept, int32_t* n_kept) {
  const int n = min(*n_tracks_p, max_tracks);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    const bool k = track_len[t] >= min_len;
    kept[t] = k ? 1 : 0;
    if (k) atomicAdd(n_kept, 1);
  }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct DetLayout {
  size_t lab, mask, part, total, bcounts, first, cnt, sums, end;
  MaskGeom g;
  int nparts;       // blocks of the maximum
  uint32_t chunk;   // words per block of the numbering passes (a multiple of the block)
  unsigned nblk;
};

DetLayout det_layout(int nx, int ny, int nz, size_t max_comp) {
  DetLayout L{};
  size_t off = 0;
  auto take = [&](size_t b) { const size_t o = off; off = align256(off + b); return o; };
  const size_t n = (size_t)nx * ny * nz, rows = (size_t)ny * nz;
  L.g = MaskGeom{nx, ny, nz, (uint32_t)((nx + 63) / 64), (uint32_t)((nx + 1) / 2), 0};
  const size_t words = rows * L.g.wpr;   // at most 2^31, as the voxels
  L.g.words = (uint32_t)words;
  const size_t per = (words + kDetBlocks - 1) / kDetBlocks;
  L.chunk = (uint32_t)((per + kDetThreads - 1) / kDetThreads * kDetThreads);
  L.nblk = (unsigned)((words + L.chunk - 1) / L.chunk);
  // (it also clears the object sums, 9 words a component)
  const size_t nb = (n + 9 * max_comp + 16 * kDetThreads - 1) / (16 * kDetThreads);
  L.nparts = (int)(nb < (size_t)kDetMaxBlocks ? nb : (size_t)kDetMaxBlocks);
  L.lab = take(rows * L.g.hx * 4);
  L.mask = take(words * 8);
  L.part = take((size_t)L.nparts * 4);
  L.total = take(4);
  L.bcounts = take((size_t)L.nblk * 4);
  L.first = take(max_comp * 4);
  L.cnt = take(max_comp * 4);
  L.sums = take(max_comp * 4 * 8);
  L.end = off;
  return L;
}

size_t link_ws_bytes(int max_n0, int max_n1) {
  return align256((size_t)max_n0 * kLinkMaxCand * 4) + align256((size_t)max_n0 * kLinkMaxCand * 8) +
         align256((size_t)max_n0 * 4) + align256((size_t)(max_n0 + max_n1) * 4);
}

ri_status hip_fail(hipError_t e, const char* what) {
  char m[256];
  snprintf(m, sizeof(m), "%s: %s", what, hipGetErrorString(e));
  return rihvr::set_error(RI_ERR_HIP, m);
}

int grid_for(size_t n) {
  const size_t b = (n + kDetThreads - 1) / kDetThreads;
  return (int)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

}  // namespace

extern "C" ri_status ri_detect_workspace_size(int32_t nx, int32_t ny, int32_t nz, int32_t max_components,
                                              size_t* bytes) {
  if (!bytes) return rihvr::set_error(RI_ERR_INVALID_ARG, "bytes is NULL");
  if (nx < 1 || ny < 1 || nz < 1 || max_components < 1)
    return rihvr::set_error(RI_ERR_INVALID_ARG, "sizes and max_components must be >= 1");
  const size_t n = (size_t)nx * ny * nz;
  if (n > ((size_t)1 << 31)) return rihvr::set_error(RI_ERR_UNSUPPORTED_SIZE, "volumes above 2^31 voxels");
  *bytes = det_layout(nx, ny, nz, (size_t)max_components).end + 256;
  return RI_OK;
}

extern "C" ri_status ri_detect(const ri_detect_params* prm, const float* x, int32_t nx, int32_t ny, int32_t nz,
                               ri_object* objects, int32_t max_objects, int32_t* counts, int32_t max_components,
                               void* ws, size_t ws_bytes, void* stream) {
  if (!prm || !x || !objects || !counts || !ws) return rihvr::set_error(RI_ERR_INVALID_ARG, "NULL argument");
  if (!(prm->rel_threshold >= 0.0) || prm->min_voxels < 1 || max_objects < 1)
    return rihvr::set_error(RI_ERR_INVALID_ARG, "rel_threshold >= 0, min_voxels >= 1, max_objects >= 1");
  size_t need = 0;
  ri_status st = ri_detect_workspace_size(nx, ny, nz, max_components, &need);
  if (st != RI_OK) return st;
  if (ws_bytes < need) return rihvr::set_error(RI_ERR_WORKSPACE_TOO_SMALL, "detect workspace too small");
  const size_t n = (size_t)nx * ny * nz;
  const DetLayout L = det_layout(nx, ny, nz, (size_t)max_components);
  char* base = reinterpret_cast<char*>(((uintptr_t)ws + 255) & ~(uintptr_t)255);
  uint32_t* lab = reinterpret_cast<uint32_t*>(base + L.lab);
  uint64_t* mask = reinterpret_cast<uint64_t*>(base + L.mask);
  float* part = reinterpret_cast<float*>(base + L.part);
  uint32_t* total = reinterpret_cast<uint32_t*>(base + L.total);
  uint32_t* bcounts = reinterpret_cast<uint32_t*>(base + L.bcounts);
  uint32_t* first = reinterpret_cast<uint32_t*>(base + L.first);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(base + L.cnt);
  double* sums = reinterpret_cast<double*>(base + L.sums);
  hipStream_t s = (hipStream_t)stream;
  const uint32_t mc = (uint32_t)max_components;
  hipError_t e;
  const dim3 b(kDetThreads), gm(grid_for((size_t)L.g.words * (64 / kDetWords)));
  hipLaunchKernelGGL(k_det_max, dim3(L.nparts), b, 0, s, x, n, part, cnt, sums, (size_t)mc);
  hipLaunchKernelGGL(k_det_mask, gm, b, 0, s, x, L.g, part, L.nparts, prm->rel_threshold, mask, lab);
  const int ps = L.g.words <= kDetSplitWords ? 3 : 0;
  hipLaunchKernelGGL(k_det_union, dim3(grid_for((size_t)L.g.words << (2 + ps))), b, 0, s, mask, L.g, ps, lab);
  hipLaunchKernelGGL(k_det_count_roots, dim3(L.nblk), b, 0, s, mask, L.g, lab, L.chunk, bcounts);
  hipLaunchKernelGGL(k_det_number, dim3(L.nblk), b, 0, s, mask, L.g, lab, L.chunk, bcounts, mc, first, total);
  const dim3 gw(grid_for((size_t)L.g.words << ps));
  hipLaunchKernelGGL(k_det_stats, gw, b, 0, s, x, mask, L.g, ps, lab, mc, cnt, sums);
  hipLaunchKernelGGL(k_det_finalize, dim3(1), dim3(kDetThreads), 0, s, cnt, sums, first, total, mc, prm->min_voxels,
                     objects, max_objects, counts);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "detect launch");
  return RI_OK;
}

extern "C" ri_status ri_link_workspace_size(int32_t max_n0, int32_t max_n1, size_t* bytes) {
  if (!bytes || max_n0 < 1 || max_n1 < 1) return rihvr::set_error(RI_ERR_INVALID_ARG, "bad link sizes");
  *bytes = link_ws_bytes(max_n0, max_n1) + 256;
  return RI_OK;
}

extern "C" ri_status ri_link(const ri_object* prev, const int32_t* n_prev, int32_t max_prev, const ri_object* cur,
                             const int32_t* n_cur, int32_t max_cur, const double spacing[3], double max_disp,
                             int32_t* link, int32_t* status, void* ws, size_t ws_bytes, void* stream) {
  if (!prev || !n_prev || !cur || !n_cur || !spacing || !link || !status || !ws)
    return rihvr::set_error(RI_ERR_INVALID_ARG, "NULL argument");
  if (max_prev < 1 || max_cur < 1 || !(max_disp > 0.0) || !(spacing[0] > 0) || !(spacing[1] > 0) || !(spacing[2] > 0))
    return rihvr::set_error(RI_ERR_INVALID_ARG, "capacities >= 1, max_disp and spacing > 0");
  if (ws_bytes < link_ws_bytes(max_prev, max_cur) + 256)
    return rihvr::set_error(RI_ERR_WORKSPACE_TOO_SMALL, "link workspace too small");
  char* base = reinterpret_cast<char*>(((uintptr_t)ws + 255) & ~(uintptr_t)255);
  LinkWs w;
  size_t off = 0;
  w.cand = reinterpret_cast<int32_t*>(base + off);
  off += align256((size_t)max_prev * kLinkMaxCand * 4);
  w.cand_d2 = reinterpret_cast<double*>(base + off);
  off += align256((size_t)max_prev * kLinkMaxCand * 8);
  w.ncand = reinterpret_cast<int32_t*>(base + off);
  off += align256((size_t)max_prev * 4);
  w.parent = reinterpret_cast<uint32_t*>(base + off);
  hipStream_t s = (hipStream_t)stream;
  hipError_t e;
  const double r2 = max_disp * max_disp;
  const int nbw = (max_prev + kDetThreads / 64 - 1) / (kDetThreads / 64);   // a wavefront per source
  hipLaunchKernelGGL(k_link_candidates, dim3(nbw), dim3(kDetThreads), 0, s, prev, n_prev, max_prev, cur, n_cur, max_cur,
                     spacing[0], spacing[1], spacing[2], r2, w, link, status);
  const int nb0 = (max_prev + kDetThreads - 1) / kDetThreads;
  hipLaunchKernelGGL(k_link_union, dim3(nb0), dim3(kDetThreads), 0, s, n_prev, max_prev, w, status);
  hipLaunchKernelGGL(k_link_roots, dim3(nb0), dim3(kDetThreads), 0, s, n_prev, max_prev, w);
  hipLaunchKernelGGL(k_link_solve, dim3(nbw), dim3(kDetThreads), 0, s, n_prev, max_prev, r2, w, link, status);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "link launch");
  return RI_OK;
}

extern "C" ri_status ri_track_update(const int32_t* link, const int32_t* n_prev, const int32_t* ids_prev,
                                     const int32_t* n_cur, int32_t max_cur, int32_t* ids_cur, int32_t* next_id,
                                     int32_t* track_len, int32_t max_tracks, void* stream) {
  if (!n_prev || !n_cur || !ids_cur || !next_id || !track_len || max_cur < 1 || max_tracks < 1)
    return rihvr::set_error(RI_ERR_INVALID_ARG, "NULL argument or capacity < 1");
  hipLaunchKernelGGL(k_track_update, dim3(1), dim3(kDetThreads), 0, (hipStream_t)stream, link, n_prev, ids_prev, n_cur,
                     max_cur, ids_cur, next_id, track_len, max_tracks);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? RI_OK : hip_fail(e, "track launch");
}

extern "C" ri_status ri_track_filter(const int32_t* track_len, const int32_t* n_tracks, int32_t max_tracks,
                                     int32_t min_len, uint8_t* kept, int32_t* n_kept, void* stream) {
  if (!track_len || !n_tracks || !kept || !n_kept || max_tracks < 1)
    return rihvr::set_error(RI_ERR_INVALID_ARG, "NULL argument or capacity < 1");
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(n_kept), (size_t)1, 0u);
  hipLaunchKernelGGL(k_track_filter, dim3((max_tracks + kDetThreads - 1) / kDetThreads), dim3(kDetThreads), 0, s,
                     track_len, n_tracks, max_tracks, min_len, kept, n_kept);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? RI_OK : hip_fail(e, "filter launch");
}
