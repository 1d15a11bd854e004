"""3x3 convolutions of launches that fill the chip (32 x 16 pixel tiles, eight
wavefronts): ragged tiles, partial channel chunks, one and two sources, each form of
the local weights, and grouped launches, against the FP64 oracle and against the
launches of single grids."""
import numpy as np
import pytest
import torch

from paper_2604_01800_amd import inputs
from oracle import net as onet
from test_gpu_net import make_net, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ppe():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_01800_amd import ppe as P
    P.lib()
    return P


# (nx, ny, levels, base, use_eta, use_spacing, nb); nb such that the finest level's
# tiles (and in the first case the next one's, with 64 output channels) fill the chip
CASES = [
    (80, 48, 3, 32, 2, 1, 64),
    (72, 40, 3, 16, 1, 1, 24),
    (48, 64, 3, 40, 0, 0, 40),
    (40, 24, 2, 24, 2, 1, 64),
    (64, 64, 3, 32, 2, 0, 64),
]


@pytest.mark.parametrize("nx,ny,L,C,eta,sp,nb", CASES)
def test_batch_of_tiles_matches_oracle(ppe, nx, ny, L, C, eta, sp, nb):
    """A batch of equal samples: every sample's output equal bit for bit (whatever tile
    and workgroup it lies in), and within the BF16 bar of test_gpu_net of the oracle."""
    cfg = onet.NetConfig(levels=L, base_channels=C, use_eta=eta, use_spacing=sp)
    g = inputs.with_ellipse(inputs.make_grid(nx, ny, 1.7, 1.3), np.random.default_rng(nx + ny))
    net, p = make_net(ppe, cfg, seed=nx * 5 + ny)
    prob = ppe.ppe_problem_create(g)
    r = (inputs.grf(g, 3, ell=0.1) * np.outer(g.hy, g.hx)).astype(np.float32)
    y = torch.zeros((nb, ny, nx), dtype=torch.float32, device="cuda")
    rd = torch.from_numpy(np.repeat(r[None], nb, 0)).cuda()
    for _ in range(3):
        y.zero_()
        ppe.ppe_net_forward(net, prob, rd, y)
        assert bool((y == y[:1]).all())
    with torch.no_grad():
        yo = onet.forward(p, cfg, g, r.astype(np.float64), g.mask, feats=onet.grid_features(g, cfg))[0].numpy()
    assert rel(y[0].cpu().numpy(), yo) <= 2e-2


@pytest.mark.parametrize("C,eta", [(32, 2), (24, 1), (32, 0)])
def test_grouped_equals_single(ppe, C, eta):
    """Forwards of grids of several sizes in grouped launches: each grid's result is that
    of its own forward, bit for bit (the K split is the grid's own; alone, the small
    grids run tiles of 16 rows)."""
    cfg = onet.NetConfig(levels=3, base_channels=C, use_eta=eta, use_spacing=1)
    net, _ = make_net(ppe, cfg, seed=11 + C)
    sizes = [(64, 48), (200, 136), (96, 320), (512, 264), (256, 256), (128, 128), (512, 264)]
    probs, rs, own = [], [], []
    for k, (nx, ny) in enumerate(sizes):
        g = inputs.with_ellipse(inputs.make_grid(nx, ny, 1.4, 1.8), np.random.default_rng(k))
        probs.append(ppe.ppe_problem_create(g))
        r = (inputs.grf(g, k, ell=0.1) * np.outer(g.hy, g.hx)).astype(np.float32)
        rs.append(torch.from_numpy(r).cuda())
        y = torch.zeros((ny, nx), dtype=torch.float32, device="cuda")
        ppe.ppe_net_forward(net, probs[-1], rs[-1], y)
        own.append(y)
    ys = [torch.zeros_like(y) for y in own]
    ppe.ppe_net_forward_batch(net, probs, rs, ys)
    torch.cuda.synchronize()
    for a, b in zip(ys, own):
        assert torch.equal(a, b)
