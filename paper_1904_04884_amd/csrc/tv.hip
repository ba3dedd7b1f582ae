// Host side of the fused-lasso proximal operator: grids, argument structs and
// launches of the TV passes (the kernels are in tv_device.h, one source file per
// fusion depth instantiates them).
#include <algorithm>
#include <vector>

#include "tv_device.h"

namespace rihvr {

// instantiated in tv_h2.hip, tv_h3.hip and tv_h4.hip
extern template void launch_tv_depth<2>(const TvSelect&, dim3, const TvPassArgs*, const BatchMap&, hipStream_t);
extern template void launch_tv_depth<3>(const TvSelect&, dim3, const TvPassArgs*, const BatchMap&, hipStream_t);
extern template void launch_tv_depth<4>(const TvSelect&, dim3, const TvPassArgs*, const BatchMap&, hipStream_t);

// Blocks of one pass: x tiles, y tiles, z chunks.  A compute unit holds one
// block, so a pass takes rounds of `fill` blocks (the units; for a frame of a
// batch its share of them) times a block's march: its planes, the margins and
// the pipeline's depth.  Of the cuts into chunks of 16 planes or more, up to
// `want` blocks, and those that still fit one round, the one of least rounds
// times march is taken; a single round counts 5/4 (its blocks run in step and
// start cold).  Prox of 20 steps at depth 3, always cutting for `want` = 1536 and
// so: 512^2 x 128 3D 2187 us (936 blocks, 4 rounds of 28 planes) and 2003 (234,
// one of 76); 256^2 x 160 920 (350, 2 of 28) and 671 (245, one of 35); 1024^2 x 64
// 4159 (1800) and 3477 (450); 512^2 x 128 in 2D stays at 936 blocks, 1242 us (one
// round of 234: 1342).  128^2 x 32, 10 steps: 24 blocks of 16 planes 208 us, 192 of
// 2 planes 118.  In a batch the frames fill the rounds together: no whole rounds,
// but a march more for the tail.
// `halo` is the tile halo of the pass (H on dual passes, H + 1 on the final).
//
// Low tiles, of 24 rows (two a lane instead of four), redo more halo but take
// about 0.6 of the time for a plane.  They are taken where their blocks fit one
// round and that outweighs the longer chunks.  Depth 3, 48 rows and 24: 64^2 x 8
// (march 11 planes and 11) 55 -> 36 us, 128^2 x 32 (11, 13) 123 -> 90, 192^2 x 48
// (13, 19) 142 -> 120, but 256^2 x 64 (19, 31) 370 -> 376; in 2D 128 x 96 x 8 (4, 4)
// 27 -> 22, but 128^2 x 32 (5, 7) 42 -> 44: lines at 0.65 and 0.75 of the march.
//
// Partial passes (fewer steps than the depth: the final pass of one step or none, every
// pass of the accelerated dual) wait for their loads, not for their steps.  In 3D they
// take the cut of least rounds times march with the margins of their own steps, a
// single round at its face value, a sixteenth of the units kept free (a nearly full
// round spills into another), and whole tiles where the leftovers of a round are split.
// In 2D, with no margin to redo, chunks of 16 planes or less.  One step, z cuts 1, 2, 4,
// 8: 512^2 x 128 3D 210, 114, 124, 135 us; 768^2 x 50 97, 129, 138, 170; 1024^2 x 64 233,
// 234, 265, 307; in 2D 214, 190, 181, 193.  So does the only pass of a prox, whose dual
// is zero (2 steps in 2D, 1024^2 x 64: 275 us with the cut of full passes, 244).
//
// With up to 2 steps such passes run at depth 2 or, where that needs no longer march (in
// 2D, where memory weighs more, a tenth longer), at depth 3: its tiles store 224 bytes of
// a row, whole 32-byte sectors, those of depth 2 232.  Two steps, depth 2 and 3: 1024^2 x
// 16 3D 82 and 75 us, 2D 73 and 67; 768^2 x 30 3D 95 and 89; but 512^2 x 24 (one round and
// two) 42 and 55.  One step in 2D: 1024 x 384 x 100 129 and 117, 1024^2 x 64 188 and 178;
// 512^2 x 128 (a march of 76 and 90) 95 and 105; without a step 1024^2 x 64 141 and 148.
struct TvGrid {
  int gx, gy, zchunk, nfull, zchunk2, nblocks, low;
  double cost;
};
// What shapes the grids of a prox's passes.
struct TvCut {
  int want, fill;
  bool alone;   // not one of several frames in a launch
  bool tv2;
  bool low;     // low tiles may be taken
  int partial;  // steps of a pass that takes fewer than its depth, else -1
  bool last;    // the final pass
};

// Thin z chunks that final_grid cuts its leftover tiles into (0: it leaves them whole).
static int leftover_chunks(int tiles, int nz, int cus) {
  if (cus <= 0 || tiles <= cus || tiles % cus == 0) return 0;
  const int k = std::min(nz, cus / (tiles % cus));
  return k < 2 ? 0 : k;
}

static TvGrid grid_of(int nx, int ny, int nz, int halo, int rows, const TvCut& c) {
  TvGrid g{};
  g.gx = (nx + (kTvRX - 2 * halo) - 1) / (kTvRX - 2 * halo);
  g.gy = (ny + (rows - 2 * halo) - 1) / (rows - 2 * halo);
  const int tiles = g.gx * g.gy, fill = std::max(1, c.fill);
  const int most = std::max(1, std::min(nz / 16, (c.want + tiles - 1) / tiles));
  const int once = std::max(1, std::min(nz, fill / tiles));
  g.cost = -1.0;
  const bool part = c.alone && c.partial >= 0;
  int n0 = 1, n1 = std::max(most, once), units = fill;
  int extra = c.tv2 ? 0 : 2 * halo, tail = halo;
  if (part) {
    extra = c.tv2 ? 0 : 2 * (c.partial + 1);
    tail = c.partial + 2;
    if (!c.tv2) {
      units -= fill / 16;
    } else if (tiles * most > fill) {
      n0 = most;
      n1 = std::min(nz, 2 * most);
    }
  }
  for (int n = n0; n <= n1; ++n) {
    const int zc = (nz + n - 1) / n, blocks = tiles * ((nz + zc - 1) / zc);
    const int march = std::min(nz, zc + extra) + tail;
    const int rounds = (blocks + units - 1) / units;
    double cost = !c.alone ? ((double)blocks / fill + 1.0) * march : (rounds == 1 && !part ? 1.25 : rounds) * (double)march;
    if (const int k = part && n == 1 && c.last ? leftover_chunks(tiles, nz, fill) : 0)
      cost = (double)(tiles / fill) * march + (nz + k - 1) / k + extra + tail;
    if (g.cost >= 0.0 && cost >= g.cost) continue;
    g.cost = cost;
    g.zchunk = zc;
    g.nblocks = blocks;
  }
  g.nfull = tiles;
  g.zchunk2 = g.zchunk;
  return g;
}
static TvGrid pass_grid(int nx, int ny, int nz, int halo, const TvCut& c) {
  const TvGrid g = grid_of(nx, ny, nz, halo, kTvRY, c);
  if (!c.low) return g;
  TvGrid h = grid_of(nx, ny, nz, halo, kTvWaves * kTvSmallQ, c);
  if (g.nblocks > c.fill || h.nblocks > c.fill || 100 * g.cost < (c.tv2 ? 75 : 65) * h.cost) return g;
  h.low = 1;
  return h;
}

// The final pass runs one 12-wave block per compute unit, so its time is
// whole rounds of `cus` blocks.  Its tiles are one voxel smaller than those of
// the dual passes; when they fill whole rounds but for a few (at 1024^2 one
// tile beyond 512), the leftover tiles are cut into thin z chunks that run
// side by side in one short extra round instead of a full one.
static TvGrid final_grid(int nx, int ny, int nz, int H, int cus, const TvCut& c) {
  TvGrid g = pass_grid(nx, ny, nz, H + 1, c);
  const int tiles = g.gx * g.gy;
  const int k = g.low || g.zchunk < nz ? 0 : leftover_chunks(tiles, nz, cus);
  if (k == 0) return g;
  const int r = tiles % cus;
  g.nfull = tiles - r;
  g.zchunk2 = (nz + k - 1) / k;
  g.nblocks = g.nfull + r * ((nz + g.zchunk2 - 1) / g.zchunk2);
  return g;
}

static int clamp_levels(int H) { return H < kTvLevelsMin ? kTvDefaultLevels : std::min(H, kTvLevelsMax); }

int prox_passes(int inner_iters, double tau, int levels, bool fgp) {
  if (!(tau > 0.0) || inner_iters <= 0) return 1;
  if (fgp) return inner_iters;        // one accelerated step per pass
  const int H = clamp_levels(levels);
  return (inner_iters + H - 1) / H;   // H dual steps per pass, the final pass included
}

// Fusion depth a prox runs with (FGP passes use the depth-2 tiles).
int prox_levels(int levels, bool fgp) { return fgp ? 2 : clamp_levels(levels); }

size_t tv_pass_args_size() { return sizeof(TvPassArgs); }

static TvCut cut_of(int blocks, int cus, int fill, int tv2, bool low) {
  return TvCut{blocks > 0 ? blocks : kTvDefaultBlocks, fill, fill >= cus, tv2 != 0, low, -1, false};
}

// A pass on full tiles: H steps at depth H, and for the final pass the steps that are
// left at a depth of as many (2 at least).
TvPassShape prox_pass_shape(int inner_iters, double tau, int levels, bool fgp, int pass) {
  const int H = prox_levels(levels, fgp), np = prox_passes(inner_iters, tau, levels, fgp);
  const int K = tau > 0.0 ? std::max(inner_iters, 0) : 0;
  TvPassShape p{};
  p.steps = fgp ? std::min(1, K) : std::min(H, K - pass * H);
  p.depth = pass == np - 1 && !fgp ? std::max(kTvLevelsMin, p.steps) : H;
  p.partial = p.steps < p.depth;
  return p;
}

// Fusion depth, dual steps, passes and cut of a prox.
struct TvProxShape {
  int H, K, npass;
  TvCut cut;
};
static TvProxShape shape_of(const ProxArgs& a) {
  const bool fgp = a.fgp != 0;
  const int H = prox_levels(a.levels, fgp);
  const bool low = H == kTvDefaultLevels && a.low && !fgp && !a.dual_bf16 && !a.rs.on;
  const double tau = a.step * a.tv;
  const int np = prox_passes(a.inner_iters, tau, a.levels, fgp);
  TvProxShape p{H, tau > 0.0 && a.inner_iters > 0 ? a.inner_iters : 0, np, cut_of(a.blocks, a.cus, a.fill, a.tv2, low)};
  if (fgp) p.cut.partial = 1;
  return p;
}
static TvGrid final_grid_of(const ProxArgs& a, const TvProxShape& h, int* depth = nullptr) {
  if (depth) *depth = h.H;
  TvCut cut = h.cut;
  cut.last = true;
  if (cut.low) {   // (low tiles exist at the default depth only, and are kept there)
    const TvGrid g = final_grid(a.nx, a.ny, a.nz, h.H, a.cus, cut);
    if (g.low) return g;
    cut.low = false;
  }
  const TvPassShape p = prox_pass_shape(a.inner_iters, a.step * a.tv, a.levels, a.fgp != 0, h.npass - 1);
  const bool only = h.npass == 1 && !a.warm && p.depth < kTvLevelsMax;
  cut.partial = p.partial || only ? p.steps : -1;
  if (depth) *depth = p.depth;
  const TvGrid g = final_grid(a.nx, a.ny, a.nz, p.depth, a.cus, cut);
  if (a.fgp || p.depth != 2 || cut.partial < 0 || !cut.alone) return g;
  const TvGrid g3 = final_grid(a.nx, a.ny, a.nz, 3, a.cus, cut);
  auto march = [&](const TvGrid& t) {
    const int rounds = (t.nblocks + cut.fill - 1) / std::max(1, cut.fill);
    return (long)rounds * (std::min(a.nz, t.zchunk + (a.tv2 ? 0 : 2 * (p.steps + 1))) + p.steps + 2);
  };
  if (10 * march(g3) > (a.tv2 && p.steps > 0 ? 11 : 10) * march(g)) return g;
  if (depth) *depth = 3;
  return g3;
}
static bool grouped(const ProxArgs& a) { return a.tv2 && a.group_planes > 0 && a.group_planes < a.nz; }

int prox_partials(const ProxArgs& pa) {
  if (!grouped(pa)) return final_grid_of(pa, shape_of(pa)).nblocks;
  ProxArgs q = pa;
  int total = 0;
  for (int z0 = 0; z0 < pa.nz; z0 += pa.group_planes) {
    q.nz = std::min(pa.group_planes, pa.nz - z0);
    total += final_grid_of(q, shape_of(q)).nblocks;
  }
  return total;
}

int tv_blocks_bound(int nx, int ny, int nz, int cus) {
  // the most tiles (the final pass's halo at the deepest fusion) times the
  // most z chunks pass_grid makes (twice nz / 16 on partial passes), or the split of final_grid (at most one
  // thin chunk per compute unit beyond the tiles), or a grid cut to fill the device
  const int h = kTvLevelsMax + 1;
  const int tx = (nx + (kTvRX - 2 * h) - 1) / (kTvRX - 2 * h);
  const int ty = (ny + (kTvRY - 2 * h) - 1) / (kTvRY - 2 * h);
  return tx * ty * std::max(1, 2 * (nz / 16)) + std::max(cus, 0);
}

int tv_group_blocks_bound(int nx, int ny, int nz, int G, int cus) {
  const int groups = (nz + G - 1) / G;
  return groups * tv_blocks_bound(nx, ny, std::min(G, nz), cus);
}

int tv_pass_zchunk(int nx, int ny, int nz, int levels, int blocks, int cus, int tv2) {
  return pass_grid(nx, ny, nz, clamp_levels(levels), cut_of(blocks, cus, cus, tv2, false)).zchunk;
}

// Whether a pass takes the sequential form (TvForm): where its steps do not fill the
// pipeline of its kernel's depth, or its blocks are short of planes.  12 steps in 3D,
// pipeline and sequential: 128^2 x 6 (6 planes) depth 3 59 and 54 us, 64^2 x 8 69 and
// 66, but 128^2 x 32 (13 planes) 97 and 100, 192^2 x 48 127 and 140; at depth 4, whose
// phases idle longer, 128^2 x 32 159 and 150, 192^2 x 48 (18 planes) 184 and 178.  The
// one pass of a prox of up to 3 steps gains more, as its dual is known to be zero: 3D, 2
// steps, 512^2 x 24 49 and 43, 512^2 x 128 218 and 186, 1024^2 x 64 356 and 324; 3 steps
// 83 and 75, 290 and 281, 396 and 376; in 2D, 3 steps, 768^2 x 30 94 and 89, 512^2 x 40 99
// and 99, but 1024^2 x 64 318 and 328; 4 steps (depth 4) 512^2 x 40 162 and 170.
static bool pass_is_seq(const ProxArgs& a, bool fin, int depth, int steps, int zchunk) {
  if (!tv_has_seq(depth, fin, a.low && !a.rs.on)) return false;
  if (steps < depth) return true;
  int most = depth > 3 ? 24 : 10;
  if (fin && depth < 4 && steps == a.inner_iters && !a.warm) most = a.tv2 ? 40 : a.nz;
  return a.low && std::min(a.nz, zchunk + (a.tv2 ? 0 : 2 * (steps + 1))) <= most;
}

// Argument structs of every pass of one prox application.  Every pass takes
// up to H dual steps; the final pass (its own tile grid, halo H + 1) also
// recovers the primal, thresholds and stores x.
int prox_pass_args(const ProxArgs& pa, void* out, int* blocks_per_pass) {
  const double tau = pa.step * pa.tv;
  const double thr = pa.step * pa.l1;
  const TvProxShape shape = shape_of(pa);
  const int H = shape.H, K = shape.K;
  const bool use_tv = K > 0, fgp = pa.fgp != 0;
  const int npass = shape.npass;
  TvPassArgs a{};
  a.v = pa.v;
  a.x = pa.x;
  for (int k = 0; k < 3; ++k) a.vol[k] = pa.vol[k];
  a.rowflag = pa.rowflag;
  a.planeflag = pa.planeflag;
  a.psum = pa.psum;
  a.ptv = pa.ptv;
  a.st = pa.st;
  a.nx = pa.nx; a.ny = pa.ny; a.nz = pa.nz;
  a.nonneg = pa.nonneg;
  a.tau = (float)tau;
  a.tv2 = pa.tv2 ? 1 : 0;
  a.dual_bf16 = pa.dual_bf16 ? 1 : 0;
  a.rs = pa.rs;
  a.c = use_tv ? (float)(1.0 / ((pa.tv2 ? 8.0 : 12.0) * tau)) : 0.f;
  a.thr = (float)thr;
  TvPassArgs* o = static_cast<TvPassArgs*>(out);
  int done = 0;
  double tk = 1.0;   // FGP: t_k of the step a pass takes
  for (int p = 0; p < npass; ++p) {
    const bool fin = p == npass - 1;
    a.depth = H;
    const TvGrid g = fin ? final_grid_of(pa, shape, &a.depth) : pass_grid(pa.nx, pa.ny, pa.nz, H, shape.cut);
    a.low = g.low;
    a.gx = g.gx;
    a.gy = g.gy;
    a.zchunk = g.zchunk;
    a.nfull = g.nfull;
    a.zchunk2 = g.zchunk2;
    a.nblocks = g.nblocks;
    if (blocks_per_pass) blocks_per_pass[p] = g.nblocks;
    const int lv = fgp ? std::min(1, K - done) : std::min(H, K - done);
    a.seq = pass_is_seq(pa, fin, a.depth, lv, g.zchunk) ? 1 : 0;
    a.levels = lv;
    a.first = (done == 0 && !pa.warm) ? 1 : 0;   // a warm dual is read by the first pass
    a.final_ = fin ? 1 : 0;
    a.keep_dual = (fin && pa.warm) ? 1 : 0;
    a.flip_npass = (pa.warm && (npass & 1)) ? npass : 0;
    a.fgp = (fgp && !fin) ? 1 : 0;
    const double tn = 0.5 * (1.0 + std::sqrt(1.0 + 4.0 * tk * tk));
    a.fgp_w = (float)((tk - 1.0) / tn);
    tk = tn;
    float* const* src = (p & 1) ? pa.pb : pa.pa;
    float* const* dst = (p & 1) ? pa.pa : pa.pb;
    float* const* src2 = (p & 1) ? pa.pb2 : pa.pa2;
    float* const* dst2 = (p & 1) ? pa.pa2 : pa.pb2;
    for (int k = 0; k < 3; ++k) {
      const bool none = pa.tv2 && k == 2;
      a.pin[k] = none ? nullptr : src[k];
      a.pout[k] = none ? nullptr : dst[k];
      a.pin2[k] = (none || !fgp) ? nullptr : src2[k];
      a.pout2[k] = (none || !fgp) ? nullptr : dst2[k];
    }
    o[p] = a;
    done += lv;
  }
  return npass;
}

// One pass of fusion depth H (FGP passes run on the depth-2 tiles).
static void launch_any(const TvSelect& k, int H, dim3 g, const TvPassArgs* a, const BatchMap& map, hipStream_t s) {
  if (k.fgp || H == 2) launch_tv_depth<2>(k, g, a, map, s);
  else if (H == 3) launch_tv_depth<3>(k, g, a, map, s);
  else launch_tv_depth<4>(k, g, a, map, s);
}
static TvSelect select_of(const TvPassArgs& a) {
  return TvSelect{false, a.final_ != 0, a.tv2 != 0, a.fgp != 0, a.dual_bf16 != 0, a.rs.on != 0, a.low != 0,
                  a.seq != 0};
}

// The per-plane 2D TV couples no planes, so its prox can run on groups of G
// planes in turn, each group's passes reading and writing a dual of G planes
// (the paper's plane-by-plane prox, with the memory of G planes instead of the
// volume).  Each group's final pass writes its objective partials after the
// previous groups' ones.
static hipError_t launch_prox_grouped(const ProxArgs& pa, int np, hipStream_t s, int* launches) {
  const int G = pa.group_planes;
  const size_t plane = (size_t)pa.nx * pa.ny;
  std::vector<TvPassArgs> args(np);
  std::vector<int> nb(np);
  int off = 0, nl = 0;
  for (int z0 = 0; z0 < pa.nz; z0 += G) {
    ProxArgs q = pa;
    q.nz = std::min(G, pa.nz - z0);
    q.group_planes = 0;
    q.rowflag = pa.rowflag ? pa.rowflag + (size_t)z0 * pa.ny : nullptr;
    q.planeflag = pa.planeflag ? pa.planeflag + z0 : nullptr;
    q.psum = pa.psum ? pa.psum + 2 * off : nullptr;
    q.ptv = pa.ptv ? pa.ptv + 2 * off : nullptr;
    if (pa.stage_group) q.x = pa.stage_group;
    const int npass = prox_pass_args(q, args.data(), nb.data());
    for (int p = 0; p < npass; ++p) {
      args[p].zoff_v = (size_t)z0 * plane;
      args[p].zoff_x = pa.stage_group ? 0 : (size_t)z0 * plane;
      launch_any(select_of(args[p]), args[p].depth, dim3(nb[p]), &args[p], BatchMap{nullptr, 0}, s);
    }
    nl += npass;
    if (pa.stage_group) {
      const hipError_t e = launch_copy_f32(pa.x + (size_t)z0 * plane, pa.stage_group, (size_t)q.nz * plane, s);
      if (e != hipSuccess) return e;
      ++nl;
    }
    off += nb[npass - 1];
  }
  if (launches) *launches = nl;
  return hipGetLastError();
}

hipError_t launch_prox(const ProxArgs& pa, hipStream_t s, int* launches) {
  const int np = shape_of(pa).npass;
  if (grouped(pa)) return launch_prox_grouped(pa, np, s, launches);
  std::vector<TvPassArgs> args(np);
  std::vector<int> nb(np);
  const int npass = prox_pass_args(pa, args.data(), nb.data());
  for (int p = 0; p < npass; ++p)
    launch_any(select_of(args[p]), args[p].depth, dim3(nb[p]), &args[p], BatchMap{nullptr, 0}, s);
  if (launches) *launches = npass;
  return hipGetLastError();
}

hipError_t launch_tv_pass_batched(int levels, bool seq, bool final_pass, bool tv2, bool fgp, bool bf16, bool sparse,
                                  const void* args, BatchMap map, int nblocks, hipStream_t s) {
  launch_any(TvSelect{true, final_pass, tv2, fgp && !final_pass, bf16, sparse, false, seq}, clamp_levels(levels),
             dim3(nblocks), static_cast<const TvPassArgs*>(args), map, s);
  return hipGetLastError();
}

}  // namespace rihvr
