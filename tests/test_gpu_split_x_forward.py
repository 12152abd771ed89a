"""Grids whose forward x transforms are split between the z-line and solve kernels
(nx = 16 and 32 with every z-line length that takes part, ny odd and even) and the
first that are not (nx = 48): Phi, the residual Jacobian action and three SBDF2
steps against the oracle, on inputs that fill every Fourier mode. Tolerance: the
FP64 path's 1e-12 (the residual's on the size of its operands)."""
import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle import gint
from oracle.befe import Befe
from oracle.grid import Grid
from paper_1804_05087_amd import SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("dims", [(16, 6, 8), (16, 9, 12), (32, 7, 24), (32, 8, 36), (16, 7, 64),
                                  (32, 6, 72), (16, 34, 8), (48, 7, 8)])
def test_parity(dims):
    from paper_1804_05087_amd import Plan
    re, dt = 400.0, 0.5
    say("split x forward", dims)
    B = Befe(Grid(*dims, *BOX), re, dt)
    P = Plan(*dims, *BOX, re, dt)
    u = synth.laminar_field(*dims) + synth.random_spectral(*dims, seed=1, scale=0.01)
    du = synth.random_spectral(*dims, seed=2)
    assert rel(to_np(P.befe_step(to_dev(u))), B.phi(u)) < TOL
    P.linearize(to_dev(u))
    phi = B.jvp(u, du, "phi")
    ref = synth.hermitian_project((phi - du) / dt)
    scale = (np.linalg.norm(phi) + np.linalg.norm(du)) / dt
    assert np.linalg.norm(to_np(P.jvp_lin(to_dev(du), SP_OP_RESIDUAL)) - ref) < TOL * scale
    P.set_scheme(1)
    P.set_steps(3)
    r = gint.sbdf2_residual(B, u, 3)
    end = np.linalg.norm(r) * 3 * 1.5 * dt + 2 * np.linalg.norm(u)
    assert np.linalg.norm(to_np(P.residual(to_dev(u))) - r) < TOL * end / (3 * 1.5 * dt)
