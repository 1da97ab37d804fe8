"""The gapless 3D step (default path of rows that are not a multiple of 64 columns): a wave takes 64 consecutive nodes
of the sequence (z, y, x).  Bitwise the row-tiled kernel (an explicit launch shape) at row lengths where a wave spans
two or three rows, wraps in y and z inside a wave, and ends past the last node.  And the 3D lattices that run on one
buffer in place though their default shape has two."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_3d_two_steps import fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny,nz,var", [(32, 3, 3, False), (33, 3, 5, True), (63, 4, 3, False), (65, 5, 7, True), (100, 33, 9, False),
                                          (193, 7, 6, True)])
def test_equals_row_tiles(q, mode, nx, ny, nz, var):
    f = fields(nx, ny, nz, nx + ny, var)
    aux = lbm.LBM_AUX_NONE if nx == 63 else lbm.LBM_AUX_LOCAL
    p = lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.03, mode, aux, nz=nz, lattice=q, phi_ref=0.4)
    tiles, flat = Solver([(p, f)]), Solver([(p, f)])
    tiles.set_launch(2, 0, tile_width=64)
    S = 0.01 * f["phi0"]
    for n, src in ((1, None), (2, [S]), (67, None)):
        tiles.step(n, S=src)
        flat.step(n, S=src)
        assert torch.equal(tiles.state_save(), flat.state_save())


@pytest.mark.parametrize("q,mode,nx,ny,nz", [(19, "f32", 68, 123, 172), (27, "f16s", 150, 130, 110)])
def test_in_place_behind_the_default_shape(q, mode, nx, ny, nz):
    """Lattices whose two buffers fit the Infinity Cache but for the unused ends of their cache lines run on one
    buffer in place; the reported shape has two.  Odd step counts, other shapes and back at one."""
    f = fields(nx, ny, nz, 7, False)
    p = lbm.make_params(nx, ny, 1.0, 1.0, 0.25, 0.03, mode, nz=nz, lattice=q, phi_ref=0.4)
    tiles, one = Solver([(p, f)]), Solver([(p, f)])
    tiles.set_launch(2, 0, tile_width=64)
    d = one.get_launch()
    assert d["stores"] == 1
    for kw in (dict(rows=1, xcd_remap=0, tile_width=256, stores=2), d, dict(rows=1, xcd_remap=1, tile_width=64, stores=1), d):
        one.step(3)
        one.set_launch(**kw)
        one.step(2)
        tiles.step(5)
        assert torch.equal(tiles.state_save(), one.state_save())
    assert one.get_launch() == d
    assert torch.equal(tiles.populations(), one.populations())
    one.step(1)
    img = one.state_save()
    one.step(4)
    one.state_load(img, 21)
    one.step(70)
    tiles.step(71)
    assert torch.equal(tiles.state_save(), one.state_save())
