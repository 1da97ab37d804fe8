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


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny,var", [(3, 16, True), (47, 18, False), (48, 33, True), (49, 40, False), (97, 64, True),
                                       (310, 131, False), (700, 517, True)])
def test_flux_form(mode, nx, ny, var):
    """The flux form's strips have 48 output columns and lag two rows per step."""
    one, two = contexts(mode, nx, ny, lbm.LBM_AUX_FLUX, var)
    S = 0.1 * dev(case(nx, ny, 3)[2]["phi0"])
    for n, src in ((4, None), (7, [S]), (71, None)):
        one.step(n, S=src)
        two.step(n, S=src)
        same(one, two)


@pytest.mark.parametrize("mode", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny,aux,var", [(3, 16, lbm.LBM_AUX_LOCAL, True), (56, 17, lbm.LBM_AUX_NONE, False),
                                           (57, 33, lbm.LBM_AUX_LOCAL, False), (230, 131, lbm.LBM_AUX_LOCAL, True),
                                           (600, 401, lbm.LBM_AUX_LOCAL, False)])
def test_walls(mode, nx, ny, aux, var):
    """Strips next to a wall reflect what crossed it, at every step of the launch, walking towards it and away.
    The flow of `case` crosses the walls, and on the smallest lattices the FP16 runs overflow within the 79
    steps: NaNs are then at the same elements (their sign bits are not defined) and every other code is equal."""
    store = {"f64": torch.float64, "f32": torch.float32, "f16s": torch.float16}[mode]
    dx, dt, f = case(nx, ny, seed=nx + ny, var=var)
    p = lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, aux, phi_ref=0.3, boundary=lbm.LBM_BC_WALLS)
    fields = {k: dev(v) for k, v in f.items()}
    one, two = Solver([(p, fields)]), Solver([(p, fields)])
    one.set_launch(2, 0, tile_width=64)
    S, pb = 0.1 * fields["phi0"], fields["phi0"] * 1.1
    for n, src in ((4, None), (5, [S]), (70, None)):
        for s in (one, two):
            s.set_dirichlet(pb)
            s.step(n, S=src)
        pb = pb * 0.9
        a, b = (s.state_save().view(store) for s in (one, two))
        nan = torch.isnan(a)
        assert torch.equal(nan, torch.isnan(b)) and torch.equal(a[~nan], b[~nan])
        if n < 70:
            same(one, two)


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32"])
@pytest.mark.parametrize("aux", [lbm.LBM_AUX_LOCAL, lbm.LBM_AUX_NONE])
def test_batch(mode, aux):
    """Every strip of every instance in one launch, with and without D and source, against serial launches;
    after another schedule and back."""
    insts, S = [], []
    for k, (nx, ny) in enumerate([(16, 16), (56, 17), (57, 64), (130, 200), (33, 48), (300, 31)]):
        dx, dt, f = case(nx, ny, seed=k, var=k % 2 == 0)
        insts.append((lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, aux), {q: dev(v) for q, v in f.items()}))
        S.append(0.1 * insts[-1][1]["phi0"] if k % 3 == 0 else None)
    one, two = Solver(insts), Solver(insts)
    one.set_batch(lbm.LBM_BATCH_SERIAL)
    batch = two.get_batch()
    for n, src in ((4, None), (7, S), (70, S), (9, None)):
        one.step(n, S=src)
        two.step(n, S=src)
        two.set_batch(lbm.LBM_BATCH_LPT, 64, 0)
        two.step(5)
        two.set_batch(**batch)
        one.step(5)
        for k in range(len(insts)):
            assert torch.equal(one.state_save(k), two.state_save(k)), k
