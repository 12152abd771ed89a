"""One Newton step of K Arnoldi iterations on grids whose dots run in groups of
different sizes (eight vectors per block on small grids, up to 32 on large ones,
four at least with the FP32 basis) and K that leaves a short last group: the
GMRES residual that the device's coefficients give equals the residual of the
step itself, r - J du by the Jacobian action, relative to |r|. The recurrence and
the true residual differ by rounding times the basis' loss of orthogonality:
1e-10 asked in FP64, 1e-5 with the FP32 basis (its vectors are accurate to 1e-7)."""
import numpy as np
import pytest

from gpu_util import BOX, say, to_dev
from paper_1804_05087_amd import SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,K", [((8, 9, 8), 1), ((8, 9, 8), 2), ((8, 9, 8), 9), ((16, 17, 16), 37),
                                    ((32, 33, 32), 41), ((48, 65, 48), 35), ((48, 65, 48), 67)])
@pytest.mark.parametrize("fp32", [False, True])
def test_recurrence_residual_is_the_residual(dims, K, fp32):
    import torch
    from paper_1804_05087_amd import Plan
    say("arnoldi", dims, K, fp32)
    P = Plan(*dims, *BOX, 400.0, 100.0)
    u = to_dev(synth.perturbation_field(*dims, *BOX, seed=0))
    x = u.clone()
    rep = P.newton_gmres(x, max_newton=1, max_krylov=K, gmres_rtol=0.0, newton_tol=0.0,
                         krylov_fp32=fp32)
    assert rep["krylov"] == [K]
    r = P.pack(P.residual(u))
    P.linearize(u)
    left = r - P.pack(P.jvp_lin((u - x).contiguous(), SP_OP_RESIDUAL))
    true = float(torch.linalg.norm(left) / torch.linalg.norm(r))
    assert np.isfinite(true)
    assert abs(true - rep["gmres_relres"][0]) < (1e-5 if fp32 else 1e-10)
