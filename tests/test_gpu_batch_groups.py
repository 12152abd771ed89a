"""Batched calls over several groups of members (a group shares its launches and
holds 256 members at most): every member equal to the single call, bit for bit,
where the count just fits one group, needs two uneven ones and leaves a short last
one; columns of the dense Jacobian over several groups equal to single actions
on unit vectors of every kind of entry."""
import numpy as np
import pytest

from gpu_util import BOX, say, to_dev
from paper_1804_05087_amd import SP_MIXED, SP_OP_PHI, SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,count,precision", [
    ((8, 9, 8), 256, 0), ((8, 9, 8), 257, 0), ((8, 9, 8), 515, SP_MIXED), ((16, 9, 6), 261, 0),
    ((54, 7, 6), 258, 0)])  # x lengths 12 and 24 (fused z-lines) and 81 (LDS transforms)
def test_groups_equal_single_calls(dims, count, precision):
    import torch
    from paper_1804_05087_amd import Plan
    say("groups", dims, count, precision)
    P = Plan(*dims, *BOX, 400.0, 10.0, precision=precision)
    few = torch.stack([to_dev(synth.perturbation_field(*dims, *BOX, seed=i)) for i in range(5)])
    u = few.repeat((count + 4) // 5, 1, 1, 1, 1)[:count].contiguous()
    u *= torch.linspace(0.5, 1.0, count, dtype=torch.float64, device=u.device)[:, None, None, None, None]
    P.linearize(few[0].contiguous())
    out = P.befe_step_batch(u)
    jb = P.jvp_lin_batch(u, SP_OP_RESIDUAL)
    half = (count + 1) // 2
    for i in sorted({0, 1, half - 1, half, count // 3, count - 2, count - 1}):
        assert torch.equal(out[i], P.befe_step(u[i].contiguous())), i
        assert torch.equal(jb[i], P.jvp_lin(u[i].contiguous(), SP_OP_RESIDUAL)), i


@pytest.mark.parametrize("op", [SP_OP_PHI, SP_OP_RESIDUAL])
def test_columns_over_several_groups(op):
    import torch
    from paper_1804_05087_amd import Plan
    dims = (8, 9, 8)
    say("columns over groups, op", op)
    P = Plan(*dims, *BOX, 400.0, 10.0)
    P.linearize(to_dev(synth.perturbation_field(*dims, *BOX, seed=3)))
    n = P.packed_n
    cols = P.jacobian_columns(op)  # all 1323
    per = 7 * 7  # reals per (component, coefficient): (0,0), m_z = 0 pairs, the rest
    for i in [0, 1, 2, 6, 7, 8, per - 1, per, 3 * per + 4, 5 * per + 30, n // 2, n - per, n - 1]:
        e = torch.zeros(n, dtype=torch.float64, device=P.device)
        e[i] = 1.0
        assert torch.equal(cols[i], P.pack(P.jvp_lin(P.unpack(e), op))), i
    assert np.isfinite(cols.cpu().numpy()).all()
