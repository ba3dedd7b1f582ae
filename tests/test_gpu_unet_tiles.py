"""U-Net kernels at the edges of their tiles: volumes smaller than a 16 x 4 x 4
box, one voxel past a box, and every channel count of the tile dispatch
(base 8 to 128), forward and gradients against the FP64 network oracle with
bfloat16 storage.  Bars as derived in test_gpu_unet: max(4e-3, 2 sens) for the
output and the loss, max(1.5e-2, 2 sens) for a gradient, with sens the oracle's
own movement under FP32-size perturbations."""
import numpy as np
import pytest

from oracle import unet as ou
from paper_1904_04884_amd import rihvr
from test_gpu_unet import flat, perturbed_bf16, rel, unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels,base,shape", [
    (1, 16, (1, 1, 1)), (1, 16, (4, 4, 16)), (1, 16, (5, 5, 17)), (1, 8, (3, 9, 33)), (1, 32, (5, 3, 20)),
    (1, 64, (2, 5, 18)), (1, 128, (3, 5, 9)), (2, 8, (2, 2, 2)), (2, 16, (6, 10, 34)), (2, 32, (10, 4, 6)),
    (2, 64, (4, 6, 18)), (3, 16, (4, 12, 20))])
def test_unet_on_ragged_tiles(torch_cuda, levels, base, shape):
    torch = torch_cuda
    rng = np.random.default_rng(levels * 1000 + base + sum(shape))
    p = ou.init_params(levels, base, rng)
    for k in p:
        p[k] = torch.tensor(p[k], dtype=torch.float32).to(torch.bfloat16).to(torch.float64).numpy()
    x = torch.tensor(rng.standard_normal(shape), dtype=torch.float32).to(torch.bfloat16).to(torch.float64).numpy()
    target = np.maximum(rng.standard_normal(shape), 0.0)
    y_ref = ou.forward(p, x, levels, base, store=ou.bf16_round)
    loss_ref, g_ref = ou.loss_and_grads(p, x, target, levels, base, store=ou.bf16_round, pos_weight=2.0)
    sens_y = rel(ou.forward(p, x, levels, base, store=perturbed_bf16(0)), y_ref)
    _, g_pert = ou.loss_and_grads(p, x, target, levels, base, store=perturbed_bf16(1), pos_weight=2.0)

    net = rihvr.UNet(levels, base, seed=1)
    net.params.copy_(torch.tensor(flat(p, levels, base), dtype=torch.float32))
    xin = torch.tensor(x, dtype=torch.float32).cuda()
    y = net.forward(xin).cpu().numpy()
    if np.linalg.norm(y_ref) > 0:
        assert rel(y, y_ref) <= max(4e-3, 2.0 * sens_y), (rel(y, y_ref), sens_y)
    else:
        assert not y.any()
    net.grads.fill_(float("nan"))   # every gradient is written
    loss = net.train_step(xin, torch.tensor(target, dtype=torch.float32).cuda(), lr=0.0, pos_weight=2.0)
    assert float(loss) == pytest.approx(loss_ref, rel=max(4e-3, 2.0 * sens_y))
    g = unflat(net.grads.cpu().numpy().astype(np.float64), levels, base, p)
    for k in g_ref:
        if np.linalg.norm(g_ref[k]) > 0:
            bar = max(1.5e-2, 2.0 * rel(g_pert[k], g_ref[k]))
            assert rel(g[k], g_ref[k]) <= bar, (k, rel(g[k], g_ref[k]), bar)
        else:
            assert not g[k].any(), k
