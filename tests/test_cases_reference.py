"""The plain 64-bit results that perf/cases.py states (dense tau systems by one LU solve,
torch's FFTs) against the oracle, every kind of case on a small grid. Tolerance: 1e-12, or
machine epsilon times the largest condition number of the per-mode systems where that is
larger; differences (. - v) / dt are held to the size of their operands."""
import numpy as np
import pytest

from oracle import gint, pack
from oracle.advect import AdvBefe
from oracle.befe import Befe
from oracle.grid import Grid
from oracle.stokes import mode_matrix
from paper_1804_05087_amd import synth
from perf import cases

DIMS, RE, DT = (8, 11, 6), 400.0, 10.0


def _case(kind, **more):
    return cases._case(kind, *DIMS, **{"re": RE, "dt": DT, **more})


def _close(a, b, dt, operands=None):
    g = Grid(*DIMS, *cases.BOX)
    cond = max(np.linalg.cond(mode_matrix(g.N, a_, b_, RE, 1.0 / dt))
               for a_, b_ in ((g.kx()[1], 0.0), (0.0, g.kz()[1])))
    tol = max(1e-12, np.finfo(float).eps * cond)
    scale = np.linalg.norm(b) if operands is None else operands
    assert np.linalg.norm(np.asarray(a) - b) < tol * scale


@pytest.mark.parametrize("kind", ["phi", "batch", "jvp", "advect", "vjp", "grad", "columns",
                                  "befe_steps", "sbdf2_steps"])
def test_exact_is_the_oracle(kind):
    more = {"batch": {"count": 2}, "columns": {"count": 40},
            "befe_steps": {"steps": 3, "scheme": 0, "dt": 0.25},
            "sbdf2_steps": {"steps": 3, "scheme": 1, "dt": 0.25}}.get(kind, {})
    c = _case("steps" if kind.endswith("steps") else kind, **more)
    dt = c["dt"]
    g = Grid(*DIMS, *cases.BOX)
    B = (AdvBefe if kind == "advect" else Befe)(g, RE, dt)
    f = {k: v.numpy() for k, v in cases._fields(c, 3).items()}
    e = cases.exact(c, 3)
    u, v = f["u"], f.get("v")
    if kind == "phi":
        _close(e, B.phi(u), dt)
    elif kind == "batch":
        for i in range(2):
            _close(e[i], B.phi(u[i]), dt)
    elif kind in ("jvp", "advect"):
        phi = B.jvp(u, v, "phi")
        _close(e, synth.hermitian_project((phi - v) / dt), dt,
               (np.linalg.norm(phi) + np.linalg.norm(v)) / dt)
    elif kind == "vjp":
        _close(e, B.vjp(u, v, "phi"), dt)
    elif kind == "grad":
        _close(e["y"], pack.pack(B.phi(u), g), dt)
        _close(e["gx"], pack.pack(B.vjp(u, v, "phi"), g), dt)
    elif kind == "columns":
        n = pack.packed_length(g)
        first = 3 * 7919 % (n - 40)
        for i in (0, 1, 17, 39):
            x = np.zeros(n)
            x[first + i] = 1.0
            d = pack.unpack(x, g)
            phi = pack.pack(B.jvp(u, d, "phi"), g)
            _close(e[i], (phi - x) / dt, dt, (np.linalg.norm(phi) + 1.0) / dt)
    else:
        sbdf2 = kind == "sbdf2_steps"
        r = (gint.sbdf2_residual if sbdf2 else gint.residual)(B, u, 3)
        span = 3 * dt * (1.5 if sbdf2 else 1.0)
        _close(e, r, dt, np.linalg.norm(r) + 2 * np.linalg.norm(u) / span)


def test_newton_has_no_plain_result():
    assert cases.exact(_case("newton", krylov=10), 1) is None
