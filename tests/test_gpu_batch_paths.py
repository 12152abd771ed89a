"""Batched calls over every kernel that takes members: each member equal to the single
call, bit for bit. Which kernels a grid runs follows its padded line lengths 3 n / 2:
6 and 9 points have no register kernel (the LDS transforms, either precision), 27, 81
and 192 have none in FP32; nx = 16 and 32 with register z-lines split the forward x
transform between the z-line and the solve (FP64; more than one group of 256 members,
so that the groups' streams take it too); long sums (ny > 68) or enough columns take
the FP64 synthesis by parities."""
import pytest

from gpu_util import BOX, say, to_dev
from paper_1804_05087_amd import SP_MIXED, SP_OP_PHI, SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,count,precision", [
    ((4, 7, 8), 5, 0), ((6, 9, 8), 300, 0), ((6, 9, 6), 7, SP_MIXED),    # LDS x-lines
    ((8, 9, 6), 6, 0), ((18, 7, 18), 9, SP_MIXED), ((54, 7, 6), 5, SP_MIXED),
    ((128, 6, 4), 3, SP_MIXED), ((12, 7, 54), 4, SP_MIXED),
    ((16, 9, 8), 300, 0), ((32, 8, 12), 260, 0),                          # split x forward
    ((8, 70, 6), 9, 0), ((6, 97, 8), 5, 0), ((96, 16, 36), 3, 0)])        # folded synthesis
def test_members_equal_single_calls(dims, count, precision):
    import torch
    from paper_1804_05087_amd import Plan
    say("batch paths", dims, count, precision)
    P = Plan(*dims, *BOX, 400.0, 10.0, precision=precision)
    few = torch.stack([to_dev(synth.laminar_field(*dims) + synth.random_spectral(*dims, seed=i, scale=0.1))
                       for i in range(3)])
    u = few.repeat((count + 2) // 3, 1, 1, 1, 1)[:count].contiguous()
    u *= torch.linspace(0.5, 1.0, count, dtype=torch.float64, device=u.device)[:, None, None, None, None]
    P.linearize(few[0].contiguous())
    out = P.befe_step_batch(u)
    jacs = [(op, P.jvp_lin_batch(u, op)) for op in (SP_OP_PHI, SP_OP_RESIDUAL)]
    half = (count + 1) // 2
    for i in sorted({0, 1, half - 1, half, count - 2, count - 1}):
        v = u[i].contiguous()
        assert torch.isfinite(torch.view_as_real(out[i])).all()
        assert torch.equal(out[i], P.befe_step(v)), i
        for op, j in jacs:
            assert torch.equal(j[i], P.jvp_lin(v, op)), (i, op)
