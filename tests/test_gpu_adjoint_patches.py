"""A segment of the reverse sweep (recomputed images and adjoint steps, four at a time on patches) against single
forward steps and lbm_adjoint_step: bitwise, for every remainder of the steps per launch and around the edges of
a patch (56 columns by 6 and by 10 rows) and the size where it changes from 12 to 16 waves."""
import pytest
import torch

from paper_2312_10316_amd import Solver, lbm
from test_gpu_fused import case, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["f64", "f64s_f32m", "f32"])
@pytest.mark.parametrize("nx,ny,steps", [(3, 3, 6), (55, 6, 4), (57, 13, 5), (64, 64, 9), (130, 41, 1), (112, 20, 11),
                                         (560, 530, 6), (561, 551, 9)])
def test_segment_equals_single_steps(mode, nx, ny, steps):
    for aux, var, src in ((lbm.LBM_AUX_LOCAL, True, True), (lbm.LBM_AUX_LOCAL, True, False), (lbm.LBM_AUX_NONE, False, True), (lbm.LBM_AUX_LOCAL, False, False)):
        dx, dt, f = case(nx, ny, seed=nx + ny, var=var)
        p = lbm.make_params(nx, ny, dx, dt, 0.25, 2e-3, mode, aux)
        fields = {k: dev(v) for k, v in f.items()}
        S = [0.1 * fields["phi0"]] if src else None
        one, two = Solver([(p, fields)]), Solver([(p, fields)])
        one.set_launch(1, 1, tile_width=256, stores=0)
        for s in (one, two):
            s.step(1, S=S)
        mdt = torch.float64 if mode == "f64" else torch.float32
        sdt = torch.float32 if mode == "f32" else torch.float64
        pitch = lbm.pitch_of(p)
        g = torch.Generator().manual_seed(steps)
        lam = torch.zeros((ny, 9, pitch), dtype=mdt)
        lam[:, :, :nx] = torch.rand((ny, 9, nx), generator=g, dtype=mdt)
        lam = lam.cuda()
        sb = lbm.lbm_state_bytes(two.ctx)
        got, tmp, images = lam.clone().ravel(), torch.zeros_like(lam).ravel(), torch.zeros(steps * sb, dtype=torch.uint8, device="cuda")
        grad = torch.rand((ny, nx), generator=g, dtype=torch.float64).cuda()
        ref_grad = grad.clone()
        images[:sb].copy_(two.state_save())
        lbm.lbm_adjoint_segment(two.ctx, 0, images, steps, got, tmp, grad)
        states = [one.state_save()]
        for _ in range(steps - 1):
            one.step(1, S=S)
            states.append(one.state_save())
        ref, out = lam.ravel(), torch.zeros_like(lam).ravel()
        for j in reversed(range(steps)):
            lbm.lbm_adjoint_step(one.ctx, 0, states[j], ref, out, ref_grad)
            ref, out = out, torch.zeros_like(lam).ravel()
        torch.cuda.synchronize()

        def nodes(t, dtype):
            return t.view(dtype)[:ny * 9 * pitch].view(ny, 9, pitch)[:, :, :nx]

        for j in range(steps):
            assert torch.equal(nodes(images[j * sb:(j + 1) * sb], sdt), nodes(states[j], sdt))
        assert torch.equal(nodes(got, mdt), nodes(ref, mdt))
        assert torch.equal(grad, ref_grad)
