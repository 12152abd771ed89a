"""The FP64 synthesis by parities (grids with enough modes, or long sums) where its
tiles and sums can go wrong: half rows that just fill a 16-row tile, leave one row
over (ny = 2^k + 1) or none in the middle (even ny), every bucket of sum lengths,
and mode counts that are no multiple of a block's 64. N(u) and the VJP (which uses
the adjoint table) against the oracle on white-noise coefficients; N's derivative
of noise carries rounding that grows with ny^2, so ny stays below 100 for N at
1e-12, and the VJP is held to 1e-12 or eps times the solve's conditioning."""
import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle import stokes
from oracle.befe import Befe
from oracle.grid import Grid
from paper_1804_05087_amd import SP_OP_PHI, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(96, 16, 36), (72, 17, 54), (54, 31, 32), (48, 32, 36),
                                  (54, 33, 32), (36, 35, 36), (8, 70, 6), (8, 96, 6), (6, 97, 8),
                                  (6, 129, 4)])
def test_parity(dims):
    from paper_1804_05087_amd import Plan
    re, dt = 400.0, 10.0
    say("synthesis fold", dims)
    nx, ny, nz = dims
    g = Grid(*dims, *BOX)
    B = Befe(g, re, dt)
    P = Plan(*dims, *BOX, re, dt)
    u = synth.perturbation_field(*dims, *BOX, seed=1)
    assert rel(to_np(P.nonlinear(to_dev(u))), B.nonlinear(u)) < 1e-12
    w = synth.random_spectral(*dims, seed=3)
    kx, kz = g.kx(), g.kz()
    cond = max(np.linalg.cond(stokes.mode_matrix(ny - 1, kx[i], kz[j], re, 1.0 / dt))
               for i, j in ((1, 0), (0, 1), (1, 1)))
    tol = max(1e-12, np.finfo(float).eps * cond)
    P.linearize(to_dev(u))
    assert rel(to_np(P.vjp_lin(to_dev(w), SP_OP_PHI)), B.vjp(u, w, "phi")) < tol
