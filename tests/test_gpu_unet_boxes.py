"""3x3x3 layers on grids with enough boxes for the high ones (eight planes, three
at 128 channels), with ragged last boxes along every axis, against the FP64
network oracle with bfloat16 storage.  Bar as in test_gpu_unet: max(4e-3, 2 sens),
sens the oracle's own movement under FP32-size perturbations."""
import numpy as np
import pytest

from oracle import unet as ou
from paper_1904_04884_amd import rihvr
from test_gpu_unet import flat, perturbed_bf16, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,shape", [(16, (42, 36, 66)), (32, (46, 66, 154)), (64, (10, 42, 90))])
def test_high_boxes(torch_cuda, base, shape):
    torch = torch_cuda
    rng = np.random.default_rng(base)
    p = ou.init_params(2, base, rng)
    for k in p:
        p[k] = torch.tensor(p[k], dtype=torch.float32).to(torch.bfloat16).to(torch.float64).numpy()
    x = torch.tensor(rng.standard_normal(shape), dtype=torch.float32).to(torch.bfloat16).to(torch.float64).numpy()
    y_ref = ou.forward(p, x, 2, base, store=ou.bf16_round)
    sens = rel(ou.forward(p, x, 2, base, store=perturbed_bf16(0)), y_ref)
    net = rihvr.UNet(2, base, seed=1)
    net.params.copy_(torch.tensor(flat(p, 2, base), dtype=torch.float32))
    y = net.forward(torch.tensor(x, dtype=torch.float32).cuda()).cpu().numpy()
    assert rel(y, y_ref) <= max(4e-3, 2.0 * sens), (rel(y, y_ref), sens)
