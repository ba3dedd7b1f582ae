// Prints, for each line "nx ny nz levels blocks fill flags group" of its input
// (flags: 1 per-plane 2D TV, 2 FGP, 4 bfloat16 dual, 8 row store, 16 low tiles
// allowed; a device of 256 units), the partials that the scalars add up, the blocks
// of the prox's final passes, the bound of both, and the planes per block of its
// first pass.  Argument: dual steps (7).
#include <cstdio>
#include <cstdlib>

#include "tv_device.h"

using namespace rihvr;

int main(int argc, char** argv) {
  const int steps = argc > 1 ? std::atoi(argv[1]) : 7;
  int nx, ny, nz, levels, blocks, fill, flags, group;
  while (std::scanf("%d %d %d %d %d %d %d %d", &nx, &ny, &nz, &levels, &blocks, &fill, &flags, &group) == 8) {
    ProxArgs a{};
    a.nx = nx; a.ny = ny; a.nz = nz;
    a.inner_iters = steps;
    a.step = 0.5; a.tv = 0.5;
    a.levels = levels; a.blocks = blocks; a.cus = 256; a.fill = fill;
    a.tv2 = flags & 1; a.fgp = (flags >> 1) & 1; a.dual_bf16 = (flags >> 2) & 1;
    a.rs.on = (flags >> 3) & 1; a.low = (flags >> 4) & 1;
    a.group_planes = group;
    const int counted = prox_partials(a);
    const int G = group > 0 ? group : nz;
    int written = 0, zchunk = 0;
    for (int z0 = 0; z0 < nz; z0 += G) {
      ProxArgs q = a;
      q.nz = std::min(G, nz - z0);
      q.group_planes = 0;
      const int np = prox_passes(q.inner_iters, q.step * q.tv, q.levels, q.fgp != 0);
      std::vector<TvPassArgs> args(np);
      std::vector<int> nb(np);
      if (prox_pass_args(q, args.data(), nb.data()) != np || !args[np - 1].final_) return 1;
      written += nb[np - 1];
      if (z0 == 0) zchunk = args[0].zchunk;
    }
    const int bound = group > 0 ? tv_group_blocks_bound(nx, ny, nz, G, a.cus) : tv_blocks_bound(nx, ny, nz, a.cus);
    std::printf("%d %d %d %d\n", counted, written, bound, zchunk);
  }
  return 0;
}
