"""The gradient-projection prox of complex and FP64 plans on grids with interior
tiles, ragged last tiles and several chunks of planes, with every remainder of
the steps per launch, and the FP64 transforms at every length: against the FP64
oracle at the bars of the other tests of these paths (1e-5 for FP32, 1e-10 for
FP64 relative L2)."""
import numpy as np
import pytest

from oracle import complex_object as co, optics, prox
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu


def geom(nx, ny, nz, **kw):
    return scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0, **kw)


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("k", (1, 3, 5, 7))
@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", ((192, 96, 9), (256, 128, 40)))
@pytest.mark.parametrize("f64", (False, True))
def test_complex_prox(torch_cuda, f64, shape, dims, k):
    torch = torch_cuda
    g = geom(*shape, tv_dims=dims, complex_object=True)
    rng = np.random.default_rng(k + dims)
    v = 0.3 * (rng.standard_normal(g.shape) + 1j * rng.standard_normal(g.shape))
    ref = co.prox_fused_lasso(v, 0.6, 0.05, 0.3, k, dims)
    p = rihvr.Plan(g, rihvr.RI_F64 if f64 else rihvr.RI_F32)
    try:
        vd = torch.from_numpy(np.stack([v.real, v.imag])).to("cuda", p.tdtype).reshape(p.shape)
        o = p.prox(vd, 0.6, 0.05, 0.3, k, nonneg=False).cpu().numpy().reshape((2,) + g.shape)
    finally:
        p.close()
    assert rel(o[0] + 1j * o[1], ref) <= (1e-10 if f64 else 1e-5)


@pytest.mark.parametrize("k", (1, 4, 5))
@pytest.mark.parametrize("dims", (2, 3))
@pytest.mark.parametrize("shape", ((192, 96, 9), (256, 128, 40)))
def test_f64_prox(torch_cuda, shape, dims, k):
    torch = torch_cuda
    g = geom(*shape, tv_dims=dims)
    v = 0.3 * np.random.default_rng(k + dims).standard_normal(g.shape)
    ref = prox.prox_fused_lasso(v, 0.6, 0.05, 0.3, k, True, dims=dims)
    p = rihvr.Plan(g, rihvr.RI_F64)
    try:
        o = p.prox(torch.from_numpy(v).cuda(), 0.6, 0.05, 0.3, k, nonneg=True).cpu().numpy()
    finally:
        p.close()
    assert rel(o, ref) <= 1e-10


@pytest.mark.parametrize("nx,ny,nz", ((16, 24, 3), (32, 16, 5), (48, 32, 1), (64, 48, 9), (96, 64, 2), (128, 96, 2),
                                      (192, 128, 7), (256, 192, 2), (384, 256, 2), (512, 384, 1), (768, 512, 1),
                                      (1024, 768, 1), (1536, 1024, 1), (2048, 1536, 1), (16, 2048, 2)))
def test_f64_transforms(torch_cuda, nx, ny, nz):
    torch = torch_cuda
    g = geom(nx, ny, nz)
    rng = np.random.default_rng(nx + ny)
    x, y = rng.standard_normal(g.shape), rng.standard_normal((ny, nx))
    p = rihvr.Plan(g, rihvr.RI_F64)
    try:
        ax = p.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        aty = p.adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    finally:
        p.close()
    assert rel(ax, optics.forward(g, x)) <= 1e-10
    assert rel(aty, optics.adjoint(g, y)) <= 1e-10
