"""Two steps per launch of one D3Q19 or D3Q27 instance (the default path where it is the faster one) against one
step per launch, bitwise: lattices of whole and ragged tiles in x (56 columns), y (14, 10 or 4 output
rows per block) and z, odd and even step counts, graph replays, sources and D
fields, and the switch between it and explicit launch shapes."""
import numpy as np
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_3d import dev

pytestmark = pytest.mark.gpu


def fields(nx, ny, nz, seed, var):
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*(2 * np.pi * np.arange(n) / n for n in (nz, ny, nx)), indexing="ij")
    f = dict(phi0=0.4 + 0.3 * np.sin(x) * np.cos(y + z) + 0.05 * rng.uniform(0, 1, (nz, ny, nx)),
             ux=0.3 * np.sin(y + 1) + 0.1, uy=0.25 * np.cos(z) * np.sin(x), uz=0.2 * np.sin(x + y) - 0.05 + 0 * z)
    f["ux"] = f["ux"] + 0 * x
    if var:
        f["D"] = 0.03 * (1 + 0.5 * rng.uniform(-1, 1, (nz, ny, nx)))
    return {k: dev(v) for k, v in f.items()}


def contexts(q, mode, nx, ny, nz, aux=lbm.LBM_AUX_LOCAL, var=False):
    f = fields(nx, ny, nz, nx + ny + nz, var)
    p = lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.03, mode, aux, nz=nz, lattice=q)
    one, two = Solver([(p, f)]), Solver([(p, f)])
    one.set_launch(2, 0, tile_width=64)
    return one, two, f


@pytest.mark.parametrize("q,mode", [(19, "f64"), (19, "f64s_f32m"), (19, "f32"), (27, "f64"), (27, "f64s_f32m"), (27, "f32")])
@pytest.mark.parametrize("nx,ny,nz,var", [(56, 300, 60, False), (100, 100, 80, True), (112, 113, 100, False), (168, 71, 70, True),
                                          (333, 150, 16, True), (333, 150, 30, False), (56, 300, 120, True)])
def test_equals_single_steps(q, mode, nx, ny, nz, var):
    aux = lbm.LBM_AUX_NONE if nx == 112 else lbm.LBM_AUX_LOCAL
    one, two, f = contexts(q, mode, nx, ny, nz, aux, var)
    S = 0.01 * f["phi0"]
    for n, src in ((2, None), (3, [S]), (68, None)):
        one.step(n, S=src)
        two.step(n, S=src)
        assert torch.equal(one.state_save(), two.state_save())
    assert torch.equal(one.populations(), two.populations())


def test_launch_shapes():
    """Explicit shapes run as asked (one buffer in place from an odd step count too), and the default one can be
    set again."""
    one, two, _ = contexts(19, "f32", 100, 100, 80)
    d = two.get_launch()
    for kw in (dict(rows=1, xcd_remap=0, tile_width=256, stores=2), dict(rows=2, xcd_remap=1, tile_width=64, stores=1), d):
        two.step(5)
        two.set_launch(**kw)
        two.step(4)
        one.step(9)
        assert torch.equal(one.state_save(), two.state_save())
    assert two.get_launch() == d
