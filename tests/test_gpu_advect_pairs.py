"""The advected step's paired real operators on the device where their layout can
go wrong: an even ny (an even number of rows), ny = 85, 86 (the rows just over the
128 pairs that one pass of a block covers), nx and nz of different sizes; the
residual action's Hermitian form; the mixed path's mean mode, which stays FP64.
Tolerances: 1e-12 (FP64, against the oracle), 2e-5 (mixed), as for the step."""
import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle import advect
from oracle.grid import Grid
from paper_1804_05087_amd import SP_MIXED, SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(12, 20, 8), (8, 85, 6), (6, 86, 8), (16, 7, 4)])
def test_parity_and_form(dims):
    from paper_1804_05087_amd import Plan
    re, dt = 400.0, 10.0
    say("advected pairs", dims)
    A = advect.AdvBefe(Grid(*dims, *BOX), re, dt)
    P = Plan(*dims, *BOX, re, dt, wall_upper=0.7, wall_lower=-0.2)
    A.wall_upper, A.wall_lower = 0.7, -0.2
    P.set_advection(True)
    u = synth.perturbation_field(*dims, *BOX, seed=2, wall_upper=0.7, wall_lower=-0.2)
    du = synth.random_admissible(*dims, *BOX, seed=3)
    assert rel(to_np(P.befe_step(to_dev(u))), A.phi(u)) < 1e-12
    j = to_np(P.jvp(to_dev(u), to_dev(du), SP_OP_RESIDUAL))
    phi = A.jvp(u, du, "phi")
    scale = (np.linalg.norm(phi) + np.linalg.norm(du)) / dt  # a difference of two fields
    assert np.linalg.norm(j - (phi - du) / dt) < 1e-12 * scale
    assert np.array_equal(synth.hermitian_project(j), j)
    P.set_precision(SP_MIXED)
    m = to_np(P.befe_step(to_dev(u)))
    assert rel(m, A.phi(u)) < 2e-5
    assert rel(m[:, 0, 0], A.phi(u)[:, 0, 0]) < 2e-5
