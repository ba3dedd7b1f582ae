"""The fused-lasso prox at the edges of its passes' grids, against the FP64
oracle: one plane, fewer planes than the pipeline is deep, grids cut to chunks
of one or a few planes, ragged last chunks, partial passes at every depth.

A prox of K <= 9 steps is K projections of sums of seven FP32 terms with
values of order 1: rel. L2 <= 1e-5, the bar of the other prox tests.  The bits
of a voxel do not depend on the grid (same operations in the same order), so
different chunkings are compared exactly."""
import numpy as np
import pytest

from oracle import prox
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu

SHAPES = [(16, 16, 1), (64, 64, 2), (64, 48, 8), (128, 96, 5), (192, 128, 33), (64, 512, 17)]


def plan_of(nx, ny, nz, dims):
    return rihvr.Plan(scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0,
                                      dz_um=50.0, tv_dims=dims))


@pytest.mark.parametrize("levels", (2, 3, 4))
@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", SHAPES)
def test_small_grids(torch_cuda, shape, dims, levels):
    torch = torch_cuda
    nx, ny, nz = shape
    plan = plan_of(nx, ny, nz, dims)
    rng = np.random.default_rng(nx + ny + nz + dims)
    v = rng.standard_normal(plan.shape).astype(np.float32)
    try:
        plan.tuning = {**plan.tuning, "tv_levels": levels}
        for k in (1, levels, levels + 1, 2 * levels + 1):
            out = plan.prox(torch.from_numpy(v).cuda(), 0.6, 0.05, 0.3, k, nonneg=k % 2 == 0).cpu().numpy()
            ref = prox.prox_fused_lasso(v.astype(np.float64), 0.6, 0.05, 0.3, k, k % 2 == 0, dims=dims)
            assert np.linalg.norm(out - ref) <= 1e-5 * np.linalg.norm(ref), k
    finally:
        plan.close()


@pytest.mark.parametrize("levels", (2, 3, 4))
def test_chunks_give_the_same_bits(torch_cuda, levels):
    """512 x 256 x 256: chunks of 64, 26 and 16 planes."""
    torch = torch_cuda
    plan = plan_of(512, 256, 256, 3)
    v = torch.randn(plan.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(levels))
    try:
        outs = []
        for blocks in (64, 512, 65536):
            plan.tuning = {**plan.tuning, "tv_levels": levels, "tv_blocks": blocks}
            outs.append(plan.prox(v, 0.6, 0.05, 0.3, 7, nonneg=True))
    finally:
        plan.close()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


def test_batch_of_small_frames(torch_cuda):
    """A frame of a batch gets its share of the device, so its chunks differ from
    the single solve's: x and the objective have the same bits all the same."""
    torch = torch_cuda
    g = scenes.Geometry(nx=64, ny=64, nz=24, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0)
    rng = np.random.default_rng(5)
    plans = [rihvr.Plan(g) for _ in range(3)]
    bs = [torch.from_numpy(rng.standard_normal((64, 64)).astype(np.float32)).cuda() for _ in plans]
    n = len(plans)
    try:
        single = [p.solve(b, 0.05, 0.05, 3, 4)[:2] for p, b in zip(plans, bs)]
        params = [p.solve_params(0.05, 0.05, 3, 4) for p in plans]
        handles = [p.handle for p in plans]
        xs = [torch.empty(p.shape, device="cuda") for p in plans]
        nbytes = rihvr.ri_workspace_size_batched(n, handles, params)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        reps = (rihvr.ri_solve_report * n)()
        st = rihvr.ri_solve_batched(n, handles, params, [b.data_ptr() for b in bs], [x.data_ptr() for x in xs],
                                    ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream, reps)
        assert st == rihvr.RI_OK
    finally:
        for p in plans:
            p.close()
    for (x, r), xb, rb in zip(single, xs, reps):
        assert torch.equal(x, xb)
        assert rb.objective == r["objective"]


@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", ((64, 64, 8), (128, 128, 32), (192, 192, 48), (96, 48, 1)))
def test_low_tiles_give_the_same_bits(torch_cuda, shape, dims):
    """Depth 3 takes low tiles on these volumes; depth 2 and 4 the full ones."""
    torch = torch_cuda
    plan = plan_of(*shape, dims)
    v = torch.randn(plan.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(shape[2]))
    try:
        outs = []
        for levels in (2, 3, 4):
            plan.tuning = {**plan.tuning, "tv_levels": levels}
            outs.append(plan.prox(v, 0.6, 0.05, 0.3, 7, nonneg=False))
    finally:
        plan.close()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
