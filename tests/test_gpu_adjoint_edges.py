"""The adjoint solve where its chains just fit their lanes: E positions per lane
of a 16-lane row hold a chain that starts at n = 0 or n = -1 up to ny = 32 E - 1.
White noise, whose highest coefficients are as large as the lowest. Tolerance:
1e-12, or machine epsilon times the largest condition number of the per-mode tau
systems where that is larger (a direct FP64 solve is backward stable only)."""
import math

import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle.befe import Befe
from oracle.grid import Grid
from oracle.stokes import mode_matrix
from paper_1804_05087_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [6, 7, 31, 32, 33, 63, 65, 66, 95, 96, 98, 127, 128])
def test_vjp_at_the_edges(ny):
    from paper_1804_05087_amd import SP_OP_PHI, SP_OP_RESIDUAL, Plan
    dims, re, dt = (8, ny, 6), 400.0, 10.0
    say("adjoint edges", dims)
    B = Befe(Grid(*dims, *BOX), re, dt)
    P = Plan(*dims, *BOX, re, dt)
    kx, kz = 2 * math.pi / BOX[0], 2 * math.pi / BOX[1]
    cond = max(np.linalg.cond(mode_matrix(ny - 1, a, b, re, 1.0 / dt))
               for a, b in ((kx, 0.0), (0.0, kz)))
    tol = max(1e-12, np.finfo(float).eps * cond)
    u = synth.perturbation_field(*dims, *BOX, seed=ny)
    w = synth.random_spectral(*dims, seed=ny + 1)
    P.linearize(to_dev(u))
    for op, name in ((SP_OP_PHI, "phi"), (SP_OP_RESIDUAL, "residual")):
        assert rel(to_np(P.vjp_lin(to_dev(w), op)), B.vjp(u, w, name)) < tol


def test_gradient_of_an_argument_changed_after_the_forward_pass():
    """The backward pass works on the state of the forward pass, bit for bit."""
    import torch
    from paper_1804_05087_amd import PhiFunction, Plan
    dims, re, dt = (8, 9, 8), 400.0, 10.0
    P = Plan(*dims, *BOX, re, dt)
    x0 = P.pack(to_dev(synth.perturbation_field(*dims, *BOX, seed=1)))
    gy = P.pack(to_dev(synth.random_spectral(*dims, seed=2)))
    grads = []
    for change in (False, True):
        x = x0.clone().requires_grad_(True)
        y = PhiFunction.apply(x, P)
        if change:
            with torch.no_grad():
                x.mul_(2.0)
        grads.append(torch.autograd.grad(y, x, gy)[0])
    assert torch.equal(*grads)
