"""Four steps per launch on strips that one wave owns (the default path of one periodic D2Q9 TRT-R instance)
against single steps.

Every node of every step runs the one-step kernel's arithmetic and the intermediate populations go
through the storage codec, so the default context must be bitwise equal to a one-step context: at strip
widths and heights around their edges (a strip has 56 output columns), lattices narrower than a wave,
every step count modulo four, and graph replays."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_fused import case, dev

pytestmark = pytest.mark.gpu


def contexts(mode, nx, ny, aux, var):
    dx, dt, f = case(nx, ny, seed=nx + 3 * ny, var=var)
    p = lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, aux, phi_ref=0.3)
    fields = {k: dev(v) for k, v in f.items()}
    one = Solver([(p, fields)])
    one.set_launch(1, 1, tile_width=256, stores=0)
    return one, Solver([(p, fields)])


def same(one, two):
    assert torch.equal(one.state_save(), two.state_save())
    assert torch.equal(one.populations(), two.populations())


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny", [(3, 16), (55, 17), (56, 33), (57, 40), (64, 64), (113, 16), (230, 131), (700, 517)])
def test_default_path_equals_single_steps(mode, nx, ny):
    for aux, var in ((lbm.LBM_AUX_LOCAL, True), (lbm.LBM_AUX_NONE, False)):
        one, two = contexts(mode, nx, ny, aux, var)
        for n in (4, 5, 3, 6, 8, 71):
            one.step(n)
            two.step(n)
            same(one, two)


@pytest.mark.parametrize("mode", ["f64", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("var", [False, True])
def test_source_and_new_velocity(mode, var):
    one, two = contexts(mode, 150, 90, lbm.LBM_AUX_LOCAL, var)
    g = torch.Generator().manual_seed(5)
    S, dS, ux, uy = (0.1 * torch.rand((90, 150), generator=g, dtype=torch.float64).cuda() for _ in range(4))
    for kw in (dict(S=[S], dSdt=[dS]), dict(ux=[ux], uy=[uy]), dict(S=[S])):
        for s in (one, two):
            s.step(13, **kw)
        same(one, two)


def test_another_launch_shape_and_back():
    """An explicit launch shape runs as asked; setting the default one again, and moving to one buffer and
    back at an odd step, keeps the state."""
    one, two = contexts("f32", 600, 520, lbm.LBM_AUX_LOCAL, True)
    d = two.get_launch()
    for kw in (dict(rows=4, xcd_remap=1, tile_width=256, fuse=2), dict(rows=1, xcd_remap=1, tile_width=256, stores=2), d):
        two.step(9)
        two.set_launch(**kw)
        two.step(9)
        one.step(18)
        same(one, two)
    assert two.get_launch() == d


@pytest.mark.parametrize("mode", ["f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny,var", [(118, 101700, False), (242, 49600, True), (3466, 3464, True)])
def test_two_columns_per_lane(mode, nx, ny, var):
    """FP16 from 12e6 nodes on an even nx: strips of 120 columns (a lattice narrower than one, two columns past
    two of them, and the smallest square one), rows around 48."""
    one, two = contexts(mode, nx, ny, lbm.LBM_AUX_LOCAL, var)
    for n in (4, 7):
        one.step(n)
        two.step(n)
        assert torch.equal(one.state_save(), two.state_save())
