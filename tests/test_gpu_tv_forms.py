"""Forms and cuts of the TV passes.  A voxel's operations do not depend on the fusion
depth, on the form of a pass (pipelined; sequential for few planes, one step or none),
on its tiles or on its z cut, so every choice gives the same bits; the small
volumes are compared with the FP64 oracle as well (rel. L2 <= 1e-5, as the other prox
tests).  Objectives: against the FP64 objective of the returned iterate, 1e-5 (transform
rounding of about 1e-6)."""
import numpy as np
import pytest

from oracle import fista, prox
from paper_1904_04884_amd import rihvr, scenes
from test_prox_grids_host import CHUNKINGS

pytestmark = pytest.mark.gpu


def geometry(nx, ny, nz, dims, **kw):
    return scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0,
                           tv_dims=dims, **kw)


def volume(torch, plan, seed):
    return torch.randn(plan.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(seed))


# 768 x 768: the last pass of one step has ten tiles more than units, cut on their own
@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", ((64, 64, 8), (128, 96, 1), (96, 96, 40), (256, 256, 17), (768, 768, 20)))
def test_depths_and_forms_give_the_same_bits(torch_cuda, shape, dims):
    torch = torch_cuda
    plan = rihvr.Plan(geometry(*shape, dims))
    v = volume(torch, plan, sum(shape))
    small = np.prod(shape) <= 1 << 17
    try:
        for k in (0, 1, 2, 3, 4, 5, 8):
            outs = []
            for levels in (2, 3, 4):
                for blocks in (64, 1536):
                    plan.tuning = {**plan.tuning, "tv_levels": levels, "tv_blocks": blocks}
                    outs.append(plan.prox(v, 0.6, 0.05, 0.3, k, nonneg=k % 2 == 0))
            assert all(torch.equal(o, outs[0]) for o in outs[1:]), k
            if small:
                ref = prox.prox_fused_lasso(v.cpu().numpy().astype(np.float64), 0.6, 0.05, 0.3, k, k % 2 == 0, dims=dims)
                assert np.linalg.norm(outs[0].cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref), k
    finally:
        plan.close()


@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape,levels,blocks", CHUNKINGS)
def test_chunkings_give_the_same_bits(torch_cuda, shape, levels, blocks, dims):
    torch = torch_cuda
    plan = rihvr.Plan(geometry(*shape, dims))
    v = volume(torch, plan, levels)
    try:
        ref = None
        for b in blocks:
            plan.tuning = {**plan.tuning, "tv_levels": levels, "tv_blocks": b}
            out = plan.prox(v, 0.6, 0.05, 0.3, 2 * levels, nonneg=True)
            ref = out if ref is None else ref
            assert torch.equal(out, ref), b
    finally:
        plan.close()


@pytest.mark.parametrize("kw", ({}, {"dual_bf16": True}))
@pytest.mark.parametrize("tv,k_in", ((0.0, 4), (0.02, 0), (0.02, 1), (0.02, 4)))
@pytest.mark.parametrize("shape,dims", (((64, 64, 8), 3), ((64, 64, 8), 2), ((768, 768, 2), 3), ((96, 48, 40), 3)))
def test_objective_after_partial_passes(torch_cuda, shape, dims, tv, k_in, kw):
    torch = torch_cuda
    g = geometry(*shape, dims, **kw)
    b = (0.3 * np.random.default_rng(sum(shape)).standard_normal((g.ny, g.nx))).astype(np.float32)
    plan = rihvr.Plan(g)
    try:
        plan.workspace(rihvr.RI_OP_SOLVE)[0].fill_(255)
        x, rep, _ = plan.solve(torch.from_numpy(b).cuda(), 0.02, tv, 3, k_in)
    finally:
        plan.close()
    x = x.cpu().numpy().astype(np.float64)
    assert (x != 0).any()
    F = fista.objective(g, x, b.astype(np.float64), 0.02, tv, tv_dims=dims)
    assert rep["objective"] == pytest.approx(F, rel=1e-5)
