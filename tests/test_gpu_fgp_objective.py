"""Objective of solves with the accelerated dual iteration, whose passes run on the
depth-2 tiles whatever depth is tuned: alone and in a batch, on volumes whose final
pass has more blocks than one of the tuned depth and on ones where it has fewer,
from a workspace full of NaN, against the FP64 objective of the returned iterate.

A x is off by about 1e-6 relative (transform rounding), the TV and l1 terms by
1e-7: 1e-5 on the objective."""
import numpy as np
import pytest

from oracle import fista
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu

L1, TV, ITERS, K_IN = 0.02, 0.02, 4, 3
SHAPES = [(48, 32, 8), (64, 64, 8), (128, 128, 8), (512, 64, 32), (512, 32, 1)]


def geometry(shape, dims, bf16=False):
    nx, ny, nz = shape
    return scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0,
                           tv_dims=dims, tv_fgp=True, dual_bf16=bf16)


def hologram(shape):
    return (0.3 * np.random.default_rng(sum(shape)).standard_normal((shape[1], shape[0]))).astype(np.float32)


def check(g, b, x, objective):
    xh = x.cpu().numpy().astype(np.float64)
    assert (xh != 0).any()
    F = fista.objective(g, xh, b.astype(np.float64), L1, TV, tv_dims=g.tv_dims)
    assert objective == pytest.approx(F, rel=1e-5)


@pytest.mark.parametrize("levels", (2, 3, 4))
@pytest.mark.parametrize("dims,bf16", ((3, False), (2, False), (3, True)))
@pytest.mark.parametrize("shape", SHAPES)
def test_single(torch_cuda, shape, dims, bf16, levels):
    torch = torch_cuda
    g, b = geometry(shape, dims, bf16), hologram(shape)
    p = rihvr.Plan(g)
    try:
        p.tuning = {**p.tuning, "tv_levels": levels}
        p.workspace(rihvr.RI_OP_SOLVE)[0].fill_(255)
        x, rep, _ = p.solve(torch.from_numpy(b).cuda(), L1, TV, ITERS, K_IN)
        check(g, b, x, rep["objective"])
    finally:
        p.close()


def test_batch(torch_cuda):
    torch = torch_cuda
    gs = [geometry(s, d) for s in SHAPES for d in (3, 2)]
    bs = [hologram((g.nx, g.ny, g.nz)) for g in gs]
    ps = [rihvr.Plan(g) for g in gs]
    try:
        for k, p in enumerate(ps):
            p.tuning = {**p.tuning, "tv_levels": 3 + k // 2 % 2}
        params = [p.solve_params(L1, TV, ITERS, K_IN) for p in ps]
        handles = [p.handle for p in ps]
        n = rihvr.ri_workspace_size_batched(len(ps), handles, params)
        ws = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
        bd = [torch.from_numpy(b).cuda() for b in bs]
        xs = [torch.empty(p.shape, device="cuda") for p in ps]
        reps = (rihvr.ri_solve_report * len(ps))()
        st = rihvr.ri_solve_batched(len(ps), handles, params, [b.data_ptr() for b in bd], [x.data_ptr() for x in xs],
                                    ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream, reps)
        assert st == rihvr.RI_OK, rihvr.ri_last_error()
        for g, b, x, r in zip(gs, bs, xs, reps):
            check(g, b, x, r.objective)
    finally:
        for p in ps:
            p.close()
