"""Several steps per launch on patches (the default path of one small D2Q9 TRT-R instance, periodic or between
walls) against single steps: bitwise, at lattice sizes around the edges of a patch (48 x 2, 56 x 6, 56 x 10, 56 x 18 and
56 x 26 output nodes) and around the sizes where the launch changes from one patch to the next, with every remainder of
the steps per launch."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_fused import case, dev
from test_gpu_strips import contexts, same

pytestmark = pytest.mark.gpu

SIZES = [(3, 3), (47, 5), (48, 4), (49, 2 * 64 + 1), (64, 64), (192, 129), (240, 102), (241, 102), (280, 306), (300, 400), (336, 426), (448, 559), (448, 660),
         (450, 732), (960, 900), (1199, 1205)]


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_patches_equal_single_steps(mode, nx, ny):
    for aux, var in ((lbm.LBM_AUX_LOCAL, True), (lbm.LBM_AUX_NONE, False), (lbm.LBM_AUX_LOCAL, False)):
        one, two = contexts(mode, nx, ny, aux, var)
        for n in (8, 9, 13, 7, 4, 75):
            one.step(n)
            two.step(n)
            same(one, two)


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (49, 7), (200, 100), (300, 240), (450, 400), (500, 500), (850, 851)])
def test_patches_between_walls(mode, nx, ny):
    dx, dt, f = case(nx, ny, seed=nx + 3 * ny, var=True)
    p = lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, lbm.LBM_AUX_LOCAL, phi_ref=0.3, boundary=lbm.LBM_BC_WALLS)
    fields = {k: dev(v) for k, v in f.items()}
    bc = torch.full((ny, nx), 0.3, dtype=torch.float64, device="cuda")
    one, two = Solver([(p, fields)]), Solver([(p, fields)])
    one.set_launch(1, 1, tile_width=256, stores=0)
    for s in (one, two):
        s.set_dirichlet(bc)
    for n in (8, 7, 12):
        one.step(n)
        two.step(n)
        a, b = one.populations(), two.populations()
        assert torch.equal(torch.nan_to_num(a, nan=-7.0), torch.nan_to_num(b, nan=-7.0))


@pytest.mark.parametrize("mode", ["f64", "f32", "f16sr"])
def test_patches_with_a_source_and_new_velocity(mode):
    one, two = contexts(mode, 150, 90, lbm.LBM_AUX_LOCAL, True)
    g = torch.Generator().manual_seed(5)
    S, dS, ux, uy = (0.1 * torch.rand((90, 150), generator=g, dtype=torch.float64).cuda() for _ in range(4))
    for kw in (dict(S=[S], dSdt=[dS]), dict(ux=[ux], uy=[uy]), dict(S=[S])):
        for s in (one, two):
            s.step(13, **kw)
        same(one, two)


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny", [(3, 24016), (57, 12017), (113, 8033), (24000, 57), (3, 28016), (57, 14017), (113, 9343)])
def test_strips_beyond_the_patches(mode, nx, ny):
    """Lattices past the patches run on strips: around one strip's 56 columns, ragged in both directions."""
    one, two = contexts(mode, nx, ny, lbm.LBM_AUX_LOCAL, True)
    for n in (4, 7, 70):
        one.step(n)
        two.step(n)
        same(one, two)
