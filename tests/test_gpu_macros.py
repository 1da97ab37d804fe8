"""Diagnostics merged by the reduction's last block into pinned host memory (lbm_macros) against the two-launch
form with a device result (lbm_macros_static): the same numbers, bit for bit, call after call."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_fused import case, dev

pytestmark = pytest.mark.gpu


def both(s, ny, nx, ref):
    phi, phi2 = (torch.empty((ny, nx), dtype=torch.float64, device="cuda") for _ in range(2))
    a = lbm.lbm_macros(s.ctx, 0, phi, ref, raise_nonfinite=False)
    b = lbm.lbm_macros_static(s.ctx, 0, phi2, ref, raise_nonfinite=False)
    torch.cuda.synchronize()
    assert a == b
    assert torch.equal(torch.nan_to_num(phi, nan=-7.0), torch.nan_to_num(phi2, nan=-7.0))
    return a


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (16, 16), (17, 16), (700, 517), (1024, 257)])
def test_one_launch_equals_two(mode, nx, ny):
    dx, dt, f = case(nx, ny, seed=nx, var=False)
    fields = {k: dev(v) for k, v in f.items()}
    s = Solver([(lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, phi_ref=0.3), fields)])
    for n in (0, 1, 3):
        s.step(n)
        for ref in (None, fields["phi0"]):
            for _ in range(3):
                both(s, ny, nx, ref)


def test_nonfinite_and_more_contexts_than_slots():
    nx, ny = 40, 30
    dx, dt, f = case(nx, ny, seed=1, var=False)
    fields = {k: dev(v) for k, v in f.items()}
    p = lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, "f32")
    want = None
    for _ in range(2):  # slots come back with their contexts
        many = [Solver([(p, fields)]) for _ in range(70)]
        for s in many:
            s.step(2)
            got = both(s, ny, nx, fields["phi0"])
            want = want or got
            assert got == want
        for s in many:
            s.close()
    s = Solver([(p, fields)])
    img = s.state_save()
    img.view(torch.float32)[5] = float("nan")
    s.state_load(img, 0)
    assert both(s, ny, nx, None)["nonfinite"] > 0
