"""Gradient-projection prox of complex and FP64 plans where a launch takes a single step
(tiles with a halo of one), at the smallest planes, ragged tiles, one plane and many
chunks, against the FP64 oracle at the bars of the other tests of these paths."""
import numpy as np
import pytest

from oracle import complex_object as co, prox
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("k", (1, 2, 4))
@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", ((16, 16, 1), (48, 24, 2), (128, 32, 33), (64, 256, 1), (256, 16, 70)))
@pytest.mark.parametrize("kind", ("complex", "complex f64", "real f64"))
def test_single_steps(torch_cuda, kind, shape, dims, k):
    torch = torch_cuda
    nx, ny, nz = shape
    cplx, f64 = kind.startswith("complex"), kind.endswith("f64")
    g = scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0,
                        tv_dims=dims, complex_object=cplx)
    rng = np.random.default_rng(nx + ny + nz + k)
    v = 0.3 * rng.standard_normal((2 if cplx else 1,) + g.shape)
    p = rihvr.Plan(g, rihvr.RI_F64 if f64 else rihvr.RI_F32)
    try:
        o = p.prox(torch.from_numpy(v).to("cuda", p.tdtype).reshape(p.shape), 0.6, 0.05, 0.3, k, nonneg=False)
        o = o.cpu().numpy().astype(np.float64).reshape(v.shape)
    finally:
        p.close()
    if cplx:
        o, ref = o[0] + 1j * o[1], co.prox_fused_lasso(v[0] + 1j * v[1], 0.6, 0.05, 0.3, k, dims)
    else:
        o, ref = o[0], prox.prox_fused_lasso(v[0], 0.6, 0.05, 0.3, k, False, dims=dims)
    assert rel(o, ref) <= (1e-10 if f64 else 1e-5)
