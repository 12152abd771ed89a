"""Padded line lengths beyond the powers of two times 3, 9: 27, 81, 162, 192, 216, 288
points in x and in z (register kernels in FP64, LDS transforms in FP32), and
z-lines of four lines per block where the number of x-lines is no multiple of
four. N(u), Phi, the residual Jacobian action and the VJP of Phi against the
oracle: 1e-12 in FP64 (ny is small, so the solve's conditioning adds nothing to
the VJP's bound), 2e-5 in mixed precision."""
import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle.befe import Befe
from oracle.grid import Grid
from paper_1804_05087_amd import SP_MIXED, SP_OP_PHI, synth

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("dims", [(18, 7, 18), (54, 8, 6), (6, 9, 54), (18, 6, 54), (108, 7, 4),
                                  (4, 7, 108), (128, 7, 6), (6, 8, 128), (144, 6, 4), (4, 6, 144),
                                  (192, 6, 4), (4, 6, 192), (18, 7, 64), (6, 7, 96)])
def test_parity(dims):
    from paper_1804_05087_amd import Plan
    re, dt = 400.0, 10.0
    say("line lengths", dims)
    B = Befe(Grid(*dims, *BOX), re, dt)
    P = Plan(*dims, *BOX, re, dt)
    u = synth.laminar_field(*dims) + synth.random_spectral(*dims, seed=1, scale=0.1)
    du = synth.random_spectral(*dims, seed=2)
    w = synth.random_spectral(*dims, seed=3)
    assert rel(to_np(P.nonlinear(to_dev(u))), B.nonlinear(u)) < TOL
    ref = B.phi(u)
    assert rel(to_np(P.befe_step(to_dev(u))), ref) < TOL
    P.linearize(to_dev(u))
    assert rel(to_np(P.jvp_lin(to_dev(du), SP_OP_PHI)), B.jvp(u, du, "phi")) < TOL
    assert rel(to_np(P.vjp_lin(to_dev(w), SP_OP_PHI)), B.vjp(u, w, "phi")) < TOL
    P.set_precision(SP_MIXED)
    assert rel(to_np(P.befe_step(to_dev(u))), ref) < 2e-5
    assert np.isfinite(to_np(P.vjp(to_dev(u), to_dev(w)))).all()
