"""One V-cycle against the oracle at the edges of the level kernels' tiles
(60 owned columns and 4 x 2, 4 or 8 rows, two-cell halos) and of the coarsest
solve's two paths (both axes of at most 128 cells, or longer). The bar is
test_gpu_mg's: a dozen FP32 stencil passes, 2e-5."""
import numpy as np
import pytest
import torch

from oracle import mg as omg
from paper_2604_01800_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,levels,nb", [
    (4, 4, 2, 1),          # a tile that is nearly all halo
    (60, 16, 2, 1),        # one full tile of columns, two of rows
    (62, 18, 2, 3),        # one column pair and one row pair more
    (120, 64, 4, 2), (124, 72, 3, 1),
    (256, 8, 2, 1), (260, 8, 2, 2),    # coarsest axis of 128 and 130 columns
    (8, 256, 2, 1), (8, 260, 2, 1),    # and of 128 and 130 rows
    (512, 272, 5, 1), (512, 272, 5, 8),  # tiles of 4 and of 8 rows on the fine level
])
def test_vcycle_at_tile_edges(nx, ny, levels, nb):
    from paper_2604_01800_amd import ppe
    rng = np.random.default_rng(nx * 1000 + ny)
    g = inputs.random_stretched_grid(nx, ny, rng)
    H = omg.Hierarchy(g, levels=levels)
    r = rng.standard_normal((nb, ny, nx))
    r = (r - r.mean(axis=(1, 2), keepdims=True)).astype(np.float32)
    z = torch.zeros((nb, ny, nx), dtype=torch.float32, device="cuda")
    prob = ppe.ppe_problem_create(g)
    ppe.ppe_apply_precond(prob, torch.from_numpy(r).cuda(), z,
                          ppe.ppe_solve_opts_default(precond=ppe.PPE_PC_MG, mg_levels=levels))
    for k in sorted({0, nb - 1}):
        want = H.apply(r[k].astype(np.float64))
        got = z[k].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - want) <= 2e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("nx,ny,levels,nb", [
    (64, 64, 4, 32), (64, 64, 4, 33),    # 256 and 264 workgroups of the first coarse launch: two and three launches
    (132, 132, 2, 4), (128, 132, 2, 5),  # two rounds of them, axes of 66 and of 64 cells: two and three launches
])
def test_vcycle_of_many_right_hand_sides(nx, ny, levels, nb):
    from paper_2604_01800_amd import ppe
    rng = np.random.default_rng(nx + 7 * ny + nb)
    g = inputs.random_stretched_grid(nx, ny, rng)
    H = omg.Hierarchy(g, levels=levels)
    r = rng.standard_normal((nb, ny, nx))
    r = (r - r.mean(axis=(1, 2), keepdims=True)).astype(np.float32)
    z = torch.zeros((nb, ny, nx), dtype=torch.float32, device="cuda")
    ppe.ppe_apply_precond(ppe.ppe_problem_create(g), torch.from_numpy(r).cuda(), z,
                          ppe.ppe_solve_opts_default(precond=ppe.PPE_PC_MG, mg_levels=levels))
    for k in (0, nb // 2, nb - 1):
        want = H.apply(r[k].astype(np.float64))
        assert np.linalg.norm(z[k].cpu().numpy() - want) <= 2e-5 * np.linalg.norm(want)
