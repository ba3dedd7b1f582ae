"""A and A^T at every transform length the library takes (each one is a radix
plan and tile shape of its own), along either axis, against the FP64 oracle:
rel. L2 <= 1e-5, the bar of the operator parity tests (FP32 transforms err by
about 1e-7 log N).  One plane per chunk, ragged chunks and many chunks reach the
sum of partial spectra with fewer and more partials than thread groups."""
import numpy as np
import pytest

from oracle import optics
from paper_1904_04884_amd import rihvr, scenes

pytestmark = pytest.mark.gpu

SIDES = (16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048)


def check(torch, nx, ny, nz, tuning=None):
    g = scenes.Geometry(nx=nx, ny=ny, nz=nz, pixel_um=5.0, wavelength_um=0.532, z0_um=5000.0, dz_um=50.0)
    rng = np.random.default_rng(nx * 7 + ny + nz)
    plan = rihvr.Plan(g)
    try:
        if tuning:
            plan.tuning = {**plan.tuning, **tuning}
        x = rng.standard_normal(g.shape).astype(np.float32)
        y = rng.standard_normal((ny, nx)).astype(np.float32)
        ax = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        aty = plan.adjoint(torch.from_numpy(y).cuda()).cpu().numpy()
    finally:
        plan.close()
    rax = optics.forward(g, x.astype(np.float64))
    raty = optics.adjoint(g, y.astype(np.float64))
    assert np.linalg.norm(ax - rax) <= 1e-5 * np.linalg.norm(rax)
    assert np.linalg.norm(aty - raty) <= 1e-5 * np.linalg.norm(raty)
    # column 0 carries the DC and Nyquist columns: compare it on its own
    f, rf = np.fft.fft2(aty)[:, :, 0], np.fft.fft2(raty)[:, :, 0]
    assert np.linalg.norm(f - rf) <= 1e-5 * np.linalg.norm(rf)


@pytest.mark.parametrize("side", SIDES)
def test_every_column_length(torch_cuda, side):
    check(torch_cuda, 32, side, 3)


@pytest.mark.parametrize("side", [s for s in SIDES if s != 24])   # rows of 24 are refused
def test_every_row_length(torch_cuda, side):
    check(torch_cuda, side, 32, 3)


@pytest.mark.parametrize("nx,ny,nz,col_blocks", [(64, 64, 1, 512), (64, 64, 37, 8192), (32, 128, 37, 16),
                                                 (48, 1024, 19, 64), (96, 96, 65, 1024), (16, 2048, 5, 8192)])
def test_partial_spectra(torch_cuda, nx, ny, nz, col_blocks):
    check(torch_cuda, nx, ny, nz, {"col_blocks": col_blocks})
