"""The Jacobian actions and the VJP at the padded line lengths 27, 81, 162, 192, 216 and
288 in either precision (register kernels in FP64, LDS transforms in FP32), in x and in
z, against the oracle. Tolerances: 1e-12 in FP64 and the mixed path's 2e-5; the residual
forms (. - v) / dt are differences, held to the size of their operands."""
import numpy as np
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle.befe import Befe
from oracle.grid import Grid
from paper_1804_05087_amd import SP_FP64, SP_MIXED, SP_OP_PHI, SP_OP_RESIDUAL, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(18, 7, 18), (54, 8, 6), (6, 9, 54), (18, 6, 54), (108, 7, 4),
                                  (4, 7, 108), (128, 7, 6), (6, 8, 128), (144, 6, 4), (4, 6, 144),
                                  (192, 6, 4), (4, 6, 192)])
@pytest.mark.parametrize("precision,tol", [(SP_FP64, 1e-12), (SP_MIXED, 2e-5)])
def test_actions(dims, precision, tol):
    from paper_1804_05087_amd import Plan
    re, dt = 400.0, 10.0
    say("line length actions", dims, precision)
    B = Befe(Grid(*dims, *BOX), re, dt)
    P = Plan(*dims, *BOX, re, dt, precision=precision)
    u = synth.laminar_field(*dims) + synth.random_spectral(*dims, seed=1, scale=0.1)
    du = synth.random_spectral(*dims, seed=2)
    w = synth.random_spectral(*dims, seed=3)
    P.linearize(to_dev(u))
    for name, v, act, ref in (("jvp", du, P.jvp_lin, B.jvp), ("vjp", w, P.vjp_lin, B.vjp)):
        phi = ref(u, v, "phi")
        e_phi = rel(to_np(act(to_dev(v), SP_OP_PHI)), phi)
        scale = (np.linalg.norm(phi) + np.linalg.norm(v)) / dt
        want = synth.hermitian_project((phi - v) / dt)
        e_res = np.linalg.norm(to_np(act(to_dev(v), SP_OP_RESIDUAL)) - want) / scale
        say(name, e_phi, e_res)
        assert e_phi < tol and e_res < tol
