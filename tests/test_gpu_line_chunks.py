"""Long x-lines whose chunks of z modes are as many as a block takes, and uneven: N(u)
against the oracle in FP64, 1e-12."""
import pytest

from gpu_util import BOX, rel, say, to_dev, to_np
from oracle.befe import Befe
from oracle.grid import Grid
from paper_1804_05087_amd import synth

pytestmark = pytest.mark.gpu


# (nx, ny, nz): padded x length and modes per block
# 144: 14 + 13, 11 + 11 + 10; 192: 7 + 7 + 7 + 6; 108: 9 + 9 + 9; 162: 11 + 11 + 10; 27: the
# same; 288: 4 + 4; 18: 9 + 9 + 9
@pytest.mark.parametrize("dims", [(96, 87, 54), (96, 33, 64), (128, 33, 54), (72, 33, 54),
                                  (108, 33, 64), (18, 40, 64), (192, 33, 16), (12, 33, 54)])
def test_nonlinear_term(dims):
    from paper_1804_05087_amd import Plan
    say("line chunks", dims)
    B = Befe(Grid(*dims, *BOX), 400.0, 10.0)
    P = Plan(*dims, *BOX, 400.0, 10.0)
    u = synth.laminar_field(*dims) + synth.random_spectral(*dims, seed=1, scale=0.1)
    assert rel(to_np(P.nonlinear(to_dev(u))), B.nonlinear(u)) < 1e-12
