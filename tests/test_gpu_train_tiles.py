"""Training gradients against the oracle's autograd at the edges of the
backward kernels' tiles: images that are no multiple of the 16-pixel tiles in
either direction, channel counts around the 16, 32, 64 and 128 channel tiles, batches
that leave splits empty. The bars are test_gpu_train's for the whole gradient
(cosine >= 0.995, relative error <= 0.1) and for the weights and biases of the layers
(cosine >= 0.98, relative error <= 0.2)."""
import numpy as np
import pytest
import torch

from oracle import net as onet
from paper_2604_01800_amd import inputs
from test_gpu_train import absolute_ok, gpu_cfg, oracle_grads, tiny_gradient

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nb,levels,base,basis,width,eta", [
    (12, 20, 1, 2, 8, 8, 8, 2),       # the narrowest network, one partial tile per level
    (40, 24, 3, 3, 8, 40, 72, 1),     # 8 to 32 channels, 1x1 layers of 40 and 72
    (36, 28, 2, 2, 24, 128, 128, 2),  # 24 and 48 channels (one and a half tiles)
    (24, 36, 2, 2, 40, 16, 128, 0),   # 40 and 80 channels, inputs of 82 and 122
    (48, 16, 5, 2, 72, 128, 16, 2),   # 72 and 144 channels: more than one 64- and 128-channel tile
])
def test_gradients_at_tile_edges(nx, ny, nb, levels, base, basis, width, eta):
    from paper_2604_01800_amd import ppe
    cfg = onet.NetConfig(levels=levels, base_channels=base, basis=basis, trunk_width=width, trunk_hidden=2,
                         phi_hidden=6, use_eta=eta)
    p = onet.round_bf16_params(cfg, onet.init_params(cfg, np.random.default_rng(nx), phi_scale=1.0))
    net = ppe.Net(gpu_cfg(ppe, cfg), seed=0)
    ppe.ppe_net_set_params(net, onet.flatten(cfg, p))
    rng = np.random.default_rng(ny)
    grids = [inputs.random_stretched_grid(nx, ny, rng, 1.0, 2.0) for _ in range(nb)]
    R = np.stack([inputs.grf(g, 50 + k, ell=0.15) * np.outer(g.hy, g.hx) for k, g in enumerate(grids)])
    R -= R.mean(axis=(1, 2), keepdims=True)
    R /= np.sqrt(np.mean(R * R, axis=(1, 2), keepdims=True))
    loss, grad = ppe.ppe_net_train_step(net, [ppe.ppe_problem_create(g) for g in grids],
                                        torch.from_numpy(R.astype(np.float32)).cuda(),
                                        ppe.ppe_train_opts_default(lr=0.0), want_grad=True)
    lo, go = oracle_grads(cfg, p, grids, R)
    assert abs(loss - lo) <= 2e-2 * lo
    a = grad.astype(np.float64)
    b = onet.flatten(cfg, {k: torch.from_numpy(v) for k, v in go.items()})
    assert float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b))) >= 0.995
    assert np.linalg.norm(a - b) <= 0.1 * np.linalg.norm(b)
    gg, grms = onet.unflatten(cfg, grad), np.linalg.norm(a) / np.sqrt(a.size)
    for name, _ in onet.param_spec(cfg):
        u, v = gg[name].numpy().reshape(-1), go[name].reshape(-1)
        if ".phi." in name or name == "head.b" or np.linalg.norm(v) == 0 or tiny_gradient(v, grms):
            assert name == "head.b" or ".phi." in name or absolute_ok(u, v, grms), name
            continue
        assert float(u @ v) >= 0.98 * np.linalg.norm(u) * np.linalg.norm(v), name
        assert np.linalg.norm(u - v) <= 0.2 * np.linalg.norm(v), name
