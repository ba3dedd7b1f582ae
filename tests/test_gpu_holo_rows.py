"""The hologram rows of an iteration in one launch (A x, residual, scalars) at
every row length and at row counts that leave a block partly idle: a solve
against the FP64 oracle at the solver tests' bar (rel. L2 1e-4), and a restarted
solve, which takes the separate launches, with the same bits where no restart
happens."""
import numpy as np
import pytest

from oracle import fista, optics
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", ((16, 16), (32, 48), (48, 32), (64, 24), (96, 64), (128, 16), (192, 32), (256, 96),
                                   (384, 16), (512, 48), (768, 16), (1024, 32), (1536, 16), (2048, 24)))
def test_solve_at_every_row_length(torch_cuda, nx, ny):
    torch = torch_cuda
    g = scenes.Geometry(nx=nx, ny=ny, nz=3, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0)
    rng = np.random.default_rng(nx + ny)
    x0 = np.maximum(rng.standard_normal(g.shape) - 1.0, 0.0)
    b = optics.forward(g, x0)
    p = rihvr.Plan(g)
    try:
        bd = torch.from_numpy(b.astype(np.float32)).cuda()
        x, rep, _ = p.solve(bd, 0.02, 0.01, 5, 3)
        xr, repr_, _ = p.solve(bd, 0.02, 0.01, 5, 3, flags=rihvr.RI_SOLVE_RESTART)
        xg, _, _ = p.solve(bd, 0.02, 0.01, 5, 3, flags=rihvr.RI_SOLVE_NO_GRAPH)
    finally:
        p.close()
    ref = fista.fista(g, b, 0.02, 0.01, 5, 3)
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(ref)
    assert torch.equal(x, xg) and torch.equal(x, xr)
    assert repr_["objective"] == pytest.approx(rep["objective"], rel=1e-12)
