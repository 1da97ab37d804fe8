"""The kernels that a default launch shape really runs on, each against single steps (an explicit launch shape):
bitwise, with the route asserted, so that a size that a rule of the dispatch has moved to another kernel fails here and
does not pass by comparing that kernel."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm

pytestmark = pytest.mark.gpu

LOCAL, FLUX, NONE = lbm.LBM_AUX_LOCAL, lbm.LBM_AUX_FLUX, lbm.LBM_AUX_NONE
STRIPS, PATCHES, PLANES, GAPLESS = lbm.LBM_ROUTE_STRIPS, lbm.LBM_ROUTE_PATCHES, lbm.LBM_ROUTE_PLANES, lbm.LBM_ROUTE_GAPLESS
TAU = 6.283185307179586


def fields(nx, ny, nz=0, var=False, seed=1):
    """A smooth flow and a rough phi0, in lattice units (dx = dt = 1)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    kw = dict(device="cuda", dtype=torch.float64)
    x = torch.arange(nx, **kw) * (TAU / nx)
    y = (torch.arange(ny, **kw) * (TAU / ny))[:, None]
    z = (torch.arange(max(nz, 1), **kw) * (TAU / max(nz, 1)))[:, None, None]
    one = torch.ones((max(nz, 1), ny, nx), **kw)
    f = {"phi0": 1 + 0.3 * torch.sin(x) * torch.cos(y + z) + 0.05 * torch.rand(one.shape, generator=g, **kw),
         "ux": 0.08 * torch.sin(y + 1) * one, "uy": 0.06 * torch.cos(x + z) * torch.sin(y) * one}
    if nz:
        f["uz"] = 0.05 * torch.sin(x + y) * one
    if var:
        f["D"] = 0.02 * (1 + 0.5 * torch.rand(one.shape, generator=g, **kw))
    return {k: (v if nz else v[0]).contiguous() for k, v in f.items()}


def compare(mode, nx, ny, aux, var, want, counts, nz=0, q=None, boundary=lbm.LBM_BC_PERIODIC, source=False):
    f = fields(nx, ny, nz, var)
    p = lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, mode, aux, phi_ref=1.0, boundary=boundary, nz=nz, lattice=q)
    one, two = Solver([(p, f)]), Solver([(p, f)])
    got = lbm.lbm_launch_route(two.ctx)
    assert {k: got[k] for k in want} == want, got
    if nz:
        one.set_launch(2, 0, tile_width=64)
    else:
        one.set_launch(1, 1, tile_width=256, stores=0)
    assert lbm.lbm_launch_route(one.ctx)["kind"] == lbm.LBM_ROUTE_TILES and lbm.lbm_launch_steps(one.ctx) == 1
    S, dS = 1e-3 * f["phi0"], 1e-4 * f["phi0"].flip(-1)
    for k, n in enumerate(counts):
        kw = dict(S=[S], dSdt=[dS]) if source and k % 2 == 0 else {}
        for s in (one, two):
            if boundary == lbm.LBM_BC_WALLS:
                s.set_dirichlet(f["phi0"] * (1 - 0.1 * k))
            s.step(n, **kw)
        assert torch.equal(one.state_save(), two.state_save()), n
    a, b = one.populations(), two.populations()
    assert torch.equal(a, b) and bool(torch.isfinite(a).all())
    one.close(), two.close()


# streaming stores, cached ones of a state within the Infinity Cache, and cached ones far beyond it
@pytest.mark.parametrize("mode,nx,ny,stores,cols", [
    ("f32", 2048, 2048, 0, 56), ("f64", 2048, 2048, 0, 56), ("f64s_f32m", 2048, 2048, 0, 56), ("f32", 2960, 2957, 1, 56),
    ("f64", 1001, 803, 1, 56), ("f64s_f32m", 1500, 1000, 1, 56), ("f32", 1500, 1201, 1, 56), ("f16s", 2311, 1103, 1, 56),
    ("f16s", 2901, 2900, 0, 56), ("f16s", 4000, 3500, 1, 120)])
def test_periodic_strips(mode, nx, ny, stores, cols):
    want = dict(kind=STRIPS, steps=4, stores=stores, cols=cols)
    for aux, var, source in ((LOCAL, False, False), (NONE, False, True), (LOCAL, True, True), (NONE, True, False)):
        compare(mode, nx, ny, aux, var, want, (4, 7, 70), source=source)


@pytest.mark.parametrize("nx,ny,var", [(120, 101700, False), (4096, 4096, True), (300, 43000, False)])
def test_stochastic_rounding_on_strips(nx, ny, var):
    compare("f16sr", nx, ny, LOCAL, var, dict(kind=STRIPS, steps=4, cols=120), (4, 7, 70))


@pytest.mark.parametrize("nx,ny,var", [(3472, 3472, False), (6100, 2000, False), (4096, 4096, False), (8192, 8192, False),
                                       (500, 30000, False)])
def test_stochastic_rounding_on_tiles(nx, ny, var):
    """From 12e6 nodes on stochastic rounding without a D field is faster on two-step tiles (3472^2: 83 us per step, on
    strips of 48 rows 111), unless the tiles hang over the lattice."""
    f = fields(nx, ny, var=var)
    s = Solver([(lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, "f16sr", phi_ref=1.0), f)])
    got = lbm.lbm_launch_route(s.ctx)
    assert (got["kind"], got["steps"]) == (lbm.LBM_ROUTE_TILES, 2), got


@pytest.mark.parametrize("nx,ny", [(3472, 3472), (5000, 5000), (6100, 2000)])
def test_rows_of_two_column_strips(nx, ny):
    """No SIMD gets a strip more than the others for the last few strips: 120-column strips in whole rounds of 1024."""
    s = Solver([(lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, "f16s", phi_ref=1.0), fields(nx, ny))])
    got = lbm.lbm_launch_route(s.ctx)
    strips = -(-nx // 120) * -(-ny // got["rows"])
    assert got["cols"] == 120 and strips / 1024 > 0.9 * -(-strips // 1024)


@pytest.mark.parametrize("mode,nx,ny,stores", [("f32", 2048, 2048, 0), ("f64", 1600, 1601, 0), ("f64s_f32m", 1600, 1601, 0),
                                               ("f16s", 2901, 2900, 0), ("f32", 1009, 1200, 1), ("f16s", 1009, 1200, 1)])
def test_flux_strips(mode, nx, ny, stores):
    for var in (False, True):
        compare(mode, nx, ny, FLUX, var, dict(kind=STRIPS, steps=4, stores=stores, cols=48), (4, 7, 70), source=var)


@pytest.mark.parametrize("mode,nx,ny,rows", [("f16s", 650, 650, (8, 12)), ("f32", 650, 650, (8, 12)), ("f16s", 64, 4000, (8, 10)), ("f64", 650, 650, (9, 12))])
def test_flux_strips_one_per_simd(mode, nx, ny, rows):
    """Two short strips on a SIMD take longer than one of twice the rows (650^2 FP16 with D, us per step: 5 rows 11.0, 9
    rows 8.8)."""
    s = Solver([(lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, mode, FLUX, phi_ref=1.0), fields(nx, ny, var=True))])
    got = lbm.lbm_launch_route(s.ctx)
    assert got["kind"] == STRIPS and rows[0] <= got["rows"] <= rows[1], got
    assert -(-nx // 48) * -(-ny // got["rows"]) <= 1024


@pytest.mark.parametrize("mode,nx,ny", [("f16s", 64, 2000), ("f32", 64, 2000), ("f64", 64, 1000), ("f64", 40, 300), ("f16s", 60000, 16)])
def test_flux_form_with_d_on_single_steps(mode, nx, ny):
    compare(mode, nx, ny, FLUX, True, dict(kind=lbm.LBM_ROUTE_TILES, steps=1), (4, 7))


@pytest.mark.parametrize("mode", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny", [(57, 12017), (1500, 1001), (2500, 1407)])
def test_strips_between_walls(mode, nx, ny):
    want = dict(kind=STRIPS, steps=4, cols=56)
    for aux, var, source in ((LOCAL, False, True), (NONE, False, False), (LOCAL, True, False), (NONE, True, True)):
        compare(mode, nx, ny, aux, var, want, (4, 7, 70), boundary=lbm.LBM_BC_WALLS, source=source)


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny,steps,rows,waves", [(64, 64, 8, 1, 16), (200, 150, 4, 1, 12), (300, 300, 4, 1, 16), (448, 400, 4, 2, 12)])
def test_periodic_patches(mode, nx, ny, steps, rows, waves):
    want = dict(kind=PATCHES, steps=steps, rows=rows, waves=waves)
    for aux, var, source in ((LOCAL, False, True), (NONE, True, True)):
        compare(mode, nx, ny, aux, var, want, (8, 13, 75), source=source)


@pytest.mark.parametrize("mode,nx,ny,boundary", [("f32", 100000, 3, lbm.LBM_BC_PERIODIC), ("f16s", 150000, 3, lbm.LBM_BC_PERIODIC),
                                                 ("f16sr", 200000, 3, lbm.LBM_BC_PERIODIC), ("f16sr", 150000, 6, lbm.LBM_BC_PERIODIC),
                                                 ("f16s", 100000, 3, lbm.LBM_BC_WALLS), ("f16sr", 100000, 4, lbm.LBM_BC_WALLS)])
def test_few_rows_stay_on_tiles(mode, nx, ny, boundary):
    """Patches of 10 output rows on a lattice of 3 took up to 1.8 times the step kernels' time."""
    compare(mode, nx, ny, LOCAL, False, dict(kind=lbm.LBM_ROUTE_TILES), (4, 7), boundary=boundary)


@pytest.mark.parametrize("mode,nx,ny", [(m, nx, ny) for m in ("f64", "f64s_f32m", "f32", "f16s", "f16sr")
                                        for nx, ny in ((2000, 3), (10000, 7), (5000, 12))]
                         + [("f32", 20000, 7), ("f16s", 20000, 7), ("f16sr", 20000, 7), ("f64s_f32m", 100000, 3)])
def test_few_rows_on_patches(mode, nx, ny):
    compare(mode, nx, ny, LOCAL, True, dict(kind=PATCHES), (8, 13))


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s", "f16sr"])
@pytest.mark.parametrize("nx,ny,steps,waves", [(64, 64, 8, 16), (200, 150, 4, 12), (400, 200, 4, 16)])
def test_patches_between_walls(mode, nx, ny, steps, waves):
    want = dict(kind=PATCHES, steps=steps, rows=1, waves=waves)
    for aux, var, source in ((LOCAL, False, True), (NONE, True, True)):
        compare(mode, nx, ny, aux, var, want, (8, 13, 75), boundary=lbm.LBM_BC_WALLS, source=source)


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny,nz", [(32, 3, 5), (33, 4, 3), (45, 7, 6), (65, 5, 7), (70, 9, 4), (90, 3, 3), (129, 5, 3)])
def test_gapless_3d(q, mode, nx, ny, nz):
    for aux, var in ((LOCAL, False), (NONE, True), (NONE, False), (LOCAL, True)):
        compare(mode, nx, ny, aux, var, dict(kind=GAPLESS, steps=1, stores=1), (1, 2, 67), nz=nz, q=q, source=var)


@pytest.mark.parametrize("aux,kind", [(NONE, lbm.LBM_ROUTE_TILES), (LOCAL, GAPLESS)])
def test_narrow_3d_lattices_beyond_the_cache(aux, kind):
    compare("f64", 36, 36, aux, True, dict(kind=kind, steps=1, stores=1), (1, 2, 67), nz=600, q=19)


def test_gapless_3d_beyond_three_quarters_of_the_cache():
    """D3Q19 FP64 without a D field: the small sizes above take four waves per SIMD, this one the compiler's choice."""
    compare("f64", 82, 82, LOCAL, False, dict(kind=GAPLESS, steps=1, stores=1), (1, 2, 67), nz=82, q=19, source=True)


@pytest.mark.parametrize("q,mode,nx,ny,nz,stores", [(19, "f32", 100, 100, 80, 1), (27, "f32", 100, 100, 80, 1),
                                                    (19, "f32", 240, 224, 64, 0), (19, "f64", 100, 100, 78, 1),
                                                    (19, "f64", 100, 100, 90, 0), (27, "f64", 100, 100, 80, 0)])
def test_two_3d_steps(q, mode, nx, ny, nz, stores):
    for aux, var in ((LOCAL, False), (NONE, True)):
        compare(mode, nx, ny, aux, var, dict(kind=PLANES, steps=2, stores=stores), (2, 3, 68), nz=nz, q=q, source=var)


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32"])
def test_batched_strips(mode):
    insts = []
    for k, (nx, ny) in enumerate([(40, 17), (130, 64), (57, 200)]):
        insts.append((lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, mode), fields(nx, ny, var=k % 2 == 0, seed=k)))
    one, two = Solver(insts), Solver(insts)
    one.set_batch(lbm.LBM_BATCH_SERIAL)
    one.set_launch(1, 1)
    got = lbm.lbm_launch_route(two.ctx)
    assert (got["kind"], got["steps"], got["stores"]) == (STRIPS, 4, 1)
    S = [1e-3 * insts[0][1]["phi0"], None, None]
    for n, src in ((4, S), (75, None)):
        one.step(n, S=src)
        two.step(n, S=src)
        for k in range(3):
            assert torch.equal(one.state_save(k), two.state_save(k))


@pytest.mark.parametrize("nx,ny,steps", [(8, 16000, 4), (3, 16001, 9), (333334, 3, 9)])
def test_adjoint_segments_that_hang_over_patches(nx, ny, steps):
    """FP64 segments that a rule keeps off the patches (all, or one of four steps) against lbm_adjoint_step."""
    f = fields(nx, ny, var=True)
    p = lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.02, "f64")
    one, two = Solver([(p, f)]), Solver([(p, f)])
    one.set_launch(1, 1, tile_width=256, stores=0)
    sb, nb = lbm.lbm_state_bytes(two.ctx), lbm.lbm_adjoint_bytes(two.ctx)
    images = torch.zeros(steps * sb, dtype=torch.uint8, device="cuda")
    images[:sb].copy_(two.state_save())
    lam, tmp, ref, out = (torch.zeros(nb, dtype=torch.uint8, device="cuda") for _ in range(4))
    grad, want = (torch.zeros((ny, nx), dtype=torch.float64, device="cuda") for _ in range(2))
    for ctx, t in ((two.ctx, lam), (one.ctx, ref)):
        lbm.lbm_adjoint_seed(ctx, 0, f["phi0"], t)
    lbm.lbm_adjoint_segment(two.ctx, 0, images, steps, lam, tmp, grad)
    states = [one.state_save()]
    for _ in range(steps - 1):
        one.step(1)
        states.append(one.state_save())
    for j in reversed(range(steps)):
        lbm.lbm_adjoint_step(one.ctx, 0, states[j], ref, out, want)
        ref, out = out, ref
    nodes = lambda t: t.view(torch.float64).view(ny, 9, -1)[:, :, :nx]
    assert torch.equal(nodes(lam), nodes(ref)) and torch.equal(grad, want)
