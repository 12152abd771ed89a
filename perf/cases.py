"""The work that a user of this library has it do, as cases that can be timed.

A case names a kind of call (`kind`), a grid (nx, ny, nz), the flow (Re, dt, the
box) and, where the call has them, its options: the precision of the actions,
the members of a batch, the columns of a Jacobian, the steps of the
time-integration operator, the length of a Krylov space. `listed()` gives the
standing ones, `draw()` more of the same ranges; `prepare()` makes what a
program holds before the call (the plan and its fields on the GPU), `run()` is
one call through the package, `work()` what the call cannot do without and
`exact()` the same result from plain torch on the host in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_05087_amd import SP_FP64, SP_MIXED, SP_OP_PHI, SP_OP_RESIDUAL, PhiFunction, Plan

BOX = (2 * math.pi / 1.14, 2 * math.pi / 2.5)  # the plane Couette box of the benchmark
LARGE_BOX = (4 * math.pi, 2 * math.pi)

# every kept Fourier size up to 128: even, with 3 n / 2 a product of 2s and 3s
FOURIER = (8, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128)


def _case(kind, nx, ny, nz, re=400.0, dt=100.0, mixed=False, large_box=False, **more):
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, re=re, dt=dt, mixed=mixed, large_box=large_box,
                **more)


def listed():
    return [
        # one step on the smallest grid of the tests and the smoke run: four launches, all latency
        dict(_case("phi", 16, 17, 16), name="phi_16x17x16"),
        # the benchmark's workload: one step at 48x65x48, Re 1000
        dict(_case("phi", 48, 65, 48, re=1000.0), name="phi_48x65x48"),
        # the large box at Re 2000, the largest grid that the benchmark runs
        dict(_case("phi", 96, 97, 96, re=2000.0, large_box=True), name="phi_96x97x96"),
        # an odd grid: an even number of Chebyshev coefficients, Fourier sizes that are no
        # multiple of 16 (padded lines of 81 and 54 points)
        dict(_case("phi", 54, 50, 36, re=700.0), name="phi_54x50x36"),
        # a wide domain: padded lines of 192 points in x and in z
        dict(_case("phi", 128, 49, 128, re=1000.0, large_box=True), name="phi_128x49x128"),
        # the matrix-vector product of a mixed-precision Newton solve about a cached state
        dict(_case("jvp", 48, 65, 48, re=1000.0, mixed=True), name="jvp_mixed_48x65x48"),
        # an adjoint search: Phi on packed vectors through autograd, forward and backward
        dict(_case("grad", 32, 33, 32), name="grad_32x33x32"),
        # one Newton step: 200 Arnoldi iterations, orthogonalisation included
        dict(_case("newton", 48, 65, 48, re=1000.0, krylov=200), name="newton_48x65x48_k200"),
        # 24 independent states (seeds, sweeps) advanced from one plan
        dict(_case("batch", 32, 33, 32, count=24), name="batch_32x33x32_24"),
        # a slice of the dense Jacobian that the spectra are computed from
        dict(_case("columns", 16, 17, 16, count=512), name="columns_16x17x16_512"),
        # the time-integration operator: the residual of 32 SBDF2 steps of 1/32
        dict(_case("steps", 32, 33, 32, dt=1.0 / 48.0, steps=32, scheme=1), name="steps_32x33x32_sbdf2"),
        # the matrix-vector product with the laminar advection in the implicit operator
        dict(_case("advect", 48, 65, 48, re=1000.0), name="advect_48x65x48"),
    ]


def _points(c):
    return c["nx"] * c["ny"] * c["nz"]


def draw(rng):
    kind = rng.choice(["phi", "phi", "phi", "jvp", "jvp", "vjp", "vjp", "grad", "batch", "columns",
                       "steps", "newton", "advect"])
    # the most points a call of this kind has: the largest listed grid for single
    # calls, less where a call does many of them or holds an operator per mode
    most = {"phi": 890_000, "jvp": 890_000, "vjp": 600_000, "grad": 400_000, "batch": 150_000,
            "columns": 20_000, "steps": 100_000, "newton": 150_000, "advect": 100_000}[kind]
    while True:
        nx, nz = rng.choice(FOURIER), rng.choice(FOURIER)
        ny = int(round(math.exp(rng.uniform(math.log(9), math.log(129)))))
        if 2_000 <= nx * ny * nz <= most and (kind != "advect" or nx * nz * ny * ny < 7_000_000):
            break
    re = float(rng.choice([200, 400, 700, 1000, 2000]))
    dt = float(rng.choice([1, 10, 100]))
    c = _case(kind, nx, ny, nz, re=re, dt=dt, large_box=rng.random() < 0.3)
    if kind in ("phi", "jvp", "vjp", "batch", "advect"):
        c["mixed"] = rng.random() < 0.3
    if kind == "batch":
        c["count"] = rng.randint(2, max(3, min(64, 2_400_000 // _points(c))))
    if kind == "columns":
        c["count"] = rng.randint(1, max(8, min(700, 2_000_000 // _points(c))))
    if kind == "steps":
        c["steps"] = rng.randint(2, 40)
        c["scheme"] = rng.randint(0, 1)
        c["dt"] = 1.0 / rng.choice([24, 32, 48])
    if kind == "newton":
        c["krylov"] = rng.randint(10, 120)
    return c


# ------------------------------------------------------------------ inputs


def _box(c):
    return LARGE_BOX if c["large_box"] else BOX


def _wavenumbers(c):
    lx, lz = _box(c)
    nx, nz = c["nx"], c["nz"]
    mx = torch.tensor([i if i < nx // 2 else i - nx for i in range(nx)], dtype=torch.float64)
    mz = torch.arange(nz // 2 + 1, dtype=torch.float64)
    return mx, mz, 2 * math.pi / lx * mx, 2 * math.pi / lz * mz


def _derivative(ny):
    """Chebyshev coefficients of p' from those of p."""
    d = torch.zeros(ny, ny, dtype=torch.float64)
    for n in range(ny):
        d[n, n + 1::2] = 2.0 * torch.arange(n + 1, ny, 2, dtype=torch.float64)
    d[0] *= 0.5
    return d


def _hermitian(a):
    """The form of a canonical field: Nyquist entries zero, the m_z = 0 plane
    Hermitian, a real (0, 0) mode."""
    nx = a.shape[-3]
    a[..., nx // 2, :, :] = 0
    a[..., -1, :] = 0
    a[..., nx // 2 + 1:, 0, :] = a[..., 1:nx // 2, 0, :].flip(-2).conj()
    a[..., 0, 0, :] = a[..., 0, 0, :].real.to(a.dtype)
    return a


def _no_slip(c, gen, energy, members=None):
    """Divergence-free fields without slip at the walls, u = curl((1 - y^2)^2 phi),
    whose spectrum falls exponentially to about 1e-4 at the edges of the grid, as
    a resolved flow's does; (1/2V) int |u|^2 = energy."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    mx, mz, kx, kz = _wavenumbers(c)
    deg = ny - 4
    n = torch.arange(deg, dtype=torch.float64)
    fall = (mx.abs()[:, None, None] / (nx / 2) + mz[None, :, None] / (nz / 2)
            + n[None, None, :] / ny)
    shape = (members or 1, 3, nx, nz // 2 + 1, deg)
    phi = torch.complex(torch.randn(shape, generator=gen, dtype=torch.float64),
                        torch.randn(shape, generator=gen, dtype=torch.float64))
    phi = _hermitian(phi * torch.exp(-9.0 * fall))
    wall = np.array([3.0 / 8.0, 0.0, -0.5, 0.0, 1.0 / 8.0])  # (1 - y^2)^2
    rows = np.zeros((ny, deg))
    for k in range(deg):
        p = np.polynomial.chebyshev.chebmul(wall, np.eye(deg)[k])[:ny]
        rows[: len(p), k] = p
    d = _derivative(ny)
    times = torch.from_numpy(rows)
    psi = torch.complex(phi.real @ times.T, phi.imag @ times.T)
    der = torch.complex(psi.real @ d.T, psi.imag @ d.T)
    ikx, ikz = 1j * kx[:, None, None], 1j * kz[None, :, None]
    u = torch.stack([der[:, 2] - ikz * psi[:, 1], ikz * psi[:, 0] - ikx * psi[:, 2],
                     ikx * psi[:, 1] - der[:, 0]], dim=1)
    u = _hermitian(u)
    s = torch.arange(ny, dtype=torch.float64)
    plus, minus = s[:, None] + s[None, :], s[:, None] - s[None, :]
    gram = torch.where(plus % 2 == 0, 1 / (1 - plus**2 + (plus % 2)) + 1 / (1 - minus**2 + (plus % 2)),
                       torch.zeros(()))
    weight = torch.where(mz == 0, 1.0, 2.0)[None, None, None, :]
    for i in range(u.shape[0]):
        e = 0.25 * sum(((p @ gram) * p).sum(-1).mul(weight[0]).sum() for p in (u[i].real, u[i].imag))
        u[i] *= math.sqrt(energy / float(e))
    return u if members else u[0]


def _fields(c, seed):
    """The host inputs of a case: states about laminar flow, directions, cotangents."""
    gen = torch.Generator().manual_seed(int(seed))
    members = c["count"] if c["kind"] == "batch" else None
    u = _no_slip(c, gen, 1e-2, members)
    u[..., 0, 0, 0, 1] += 1.0  # U = y e_x
    f = {"u": u}
    if c["kind"] in ("jvp", "vjp", "advect", "grad"):
        f["v"] = _no_slip(c, gen, 0.5)
    return f


def _packed_order(c):
    """Positions (in the canonical field) and parts of the packed real vector."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    nzh = nz // 2 + 1
    pairs = [(0, 0, 0)]
    pairs += [(i, 0, part) for i in range(1, nx // 2) for part in (0, 1)]
    pairs += [(i, j, part) for j in range(1, nz // 2) for i in range(nx) if i != nx // 2
              for part in (0, 1)]
    p = np.array(pairs)
    one = (p[:, 0] * nzh + p[:, 1]) * ny
    at = (np.arange(3)[:, None, None] * (nx * nzh * ny) + np.arange(ny)[None, :, None] + one)
    return torch.from_numpy(2 * at + p[:, 2]).reshape(-1)


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    f = {k: v.to(dev) for k, v in _fields(c, seed).items()}
    lx, lz = _box(c)
    plan = Plan(c["nx"], c["ny"], c["nz"], lx, lz, c["re"], c["dt"],
                precision=SP_MIXED if c["mixed"] else SP_FP64, device=dev)
    s = dict(f, kind=c["kind"], plan=plan, case=c)
    if c["kind"] == "steps":
        plan.set_scheme(c["scheme"])
        plan.set_steps(c["steps"])
    if c["kind"] == "advect":
        plan.set_advection(True)
    if c["kind"] in ("jvp", "vjp", "columns", "advect"):
        plan.linearize(s["u"])
    if c["kind"] == "columns":
        # the slice starts at a place of its own for every seed
        s["first"] = int(seed) * 7919 % max(1, plan.packed_n - c["count"])
    if c["kind"] == "grad":
        s["x"] = plan.pack(s.pop("u"))
        s["gy"] = plan.pack(s.pop("v"))
    return s


def run(state):
    s = state
    plan, kind = s["plan"], s["kind"]
    if kind == "phi":
        return plan.befe_step(s["u"])
    if kind == "jvp" or kind == "advect":
        return plan.jvp_lin(s["v"], SP_OP_RESIDUAL)
    if kind == "vjp":
        return plan.vjp_lin(s["v"], SP_OP_PHI)
    if kind == "grad":
        x = s["x"].detach().requires_grad_(True)
        y = PhiFunction.apply(x, plan)
        (gx,) = torch.autograd.grad(y, x, s["gy"])
        return {"y": y.detach(), "gx": gx}
    if kind == "batch":
        return plan.befe_step_batch(s["u"])
    if kind == "columns":
        return plan.jacobian_columns(SP_OP_RESIDUAL, s["first"], s["case"]["count"])
    if kind == "steps":
        return plan.residual(s["u"])
    u = s["u"].clone()
    rep = plan.newton_gmres(u, max_newton=1, max_krylov=s["case"]["krylov"], gmres_rtol=0.0,
                            newton_tol=0.0)
    return {"u": u, "res_norm": np.array(rep["res_norm"])}


# ------------------------------------------------------------------ what a call cannot do without


def work(case):
    c = case
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    field = 3 * nx * (nz // 2 + 1) * ny * 16
    px, pz = 3 * nx // 2, 3 * nz // 2
    # real transforms of nine fields over every padded plane, products, y-transforms
    # by the fast cosine transform and about 60 operations per coefficient of the solve
    fft = 9 * ny * 2.5 * px * pz * math.log2(px * pz)
    step = fft + 9 * ny * px * pz + 8 * 2.5 * nx * nz * ny * math.log2(2 * ny) + 60 * 3 * nx * nz * ny
    base = 6 * ny * px * pz * (4 if c["mixed"] else 8)
    if c["kind"] == "phi":
        return {"bytes": 2 * field, "flops": step}
    if c["kind"] in ("jvp", "vjp"):
        return {"bytes": 2 * field + base, "flops": 1.2 * step}
    if c["kind"] == "grad":
        return {"bytes": 4 * field, "flops": 2.9 * step}
    if c["kind"] == "batch":
        return {"bytes": 2 * field * c["count"], "flops": step * c["count"]}
    if c["kind"] == "columns":
        return {"bytes": base + field * c["count"], "flops": 1.2 * step * c["count"]}
    if c["kind"] == "steps":
        return {"bytes": 2 * field, "flops": step * c["steps"]}
    if c["kind"] == "advect":
        # each mode's dense solution operator, a real matrix shared by m_x and -m_x
        entries = 9.0 * (ny - 2) * ny * (nx // 2 + 1) * (nz // 2)
        return {"bytes": 2 * field + base + entries * (4 if c["mixed"] else 8),
                "flops": 1.2 * step + 8 * entries}
    k = c["krylov"]
    vector = 3 * ny * (nx - 1) * (nz - 1) * 8
    return {"bytes": vector * k * (k + 1) / 2 + k * base, "flops": 1.2 * step * k + 4.0 * vector / 8 * k * k}


# ------------------------------------------------------------------ the same results, from plain torch on the host


class _Reference:
    """The step of the paper's eq. befe for one grid in 64 bits: dense Chebyshev
    matrices, torch's FFTs on the 3/2 grid, dense tau systems per mode."""

    def __init__(self, c, advect=False):
        self.c = c
        nx, ny, nz = c["nx"], c["ny"], c["nz"]
        self.nx, self.ny, self.nz = nx, ny, nz
        self.px, self.pz = 3 * nx // 2, 3 * nz // 2
        self.inv_dt = 1.0 / c["dt"]
        _, _, self.kx, self.kz = _wavenumbers(c)
        th = math.pi * torch.arange(ny, dtype=torch.float64) / (ny - 1)
        self.T = torch.cos(th[:, None] * torch.arange(ny, dtype=torch.float64)[None, :])
        self.Tinv = torch.linalg.inv(self.T)
        self.D = _derivative(ny)
        self.advect = advect
        if advect:
            self._advected_operators()
        else:
            self._operators()

    # ---- fields and their products

    def _y(self, m, a):
        return torch.complex(a.real @ m.T, a.imag @ m.T)

    def _physical(self, a):
        """Values on the padded grid [..., y, px, pz] of coefficients [..., nx, nzh, ny]."""
        nx, nz = self.nx, self.nz
        v = self._y(self.T, a).movedim(-1, -3)
        full = torch.zeros(*v.shape[:-2], self.px, self.pz // 2 + 1, dtype=v.dtype)
        full[..., :nx // 2, :nz // 2] = v[..., :nx // 2, :nz // 2]
        full[..., self.px - nx // 2 + 1:, :nz // 2] = v[..., nx // 2 + 1:, :nz // 2]
        return torch.fft.irfft2(full, s=(self.px, self.pz), norm="forward")

    def _spectral(self, f):
        nx, nz = self.nx, self.nz
        h = torch.fft.rfft2(f, norm="forward")
        v = torch.zeros(*h.shape[:-2], nx, nz // 2 + 1, dtype=h.dtype)
        v[..., :nx // 2, :nz // 2] = h[..., :nx // 2, :nz // 2]
        v[..., nx // 2 + 1:, :nz // 2] = h[..., self.px - nx // 2 + 1:, :nz // 2]
        return self._y(self.Tinv, v.movedim(-3, -1))

    def _curl(self, a):
        d = self._y(self.D, a)
        ikx, ikz = 1j * self.kx[:, None, None], 1j * self.kz[None, :, None]
        u, v, w = a.unbind(-4)
        return torch.stack([d.select(-4, 2) - ikz * v, ikz * u - ikx * w, ikx * v - d.select(-4, 0)], dim=-4)

    @staticmethod
    def _cross(a, b):
        return torch.stack([a[..., 1, :, :, :] * b[..., 2, :, :, :] - a[..., 2, :, :, :] * b[..., 1, :, :, :],
                            a[..., 2, :, :, :] * b[..., 0, :, :, :] - a[..., 0, :, :, :] * b[..., 2, :, :, :],
                            a[..., 0, :, :, :] * b[..., 1, :, :, :] - a[..., 1, :, :, :] * b[..., 0, :, :, :]],
                           dim=-4)

    def nonlinear(self, u):
        return self._spectral(self._cross(self._physical(u), self._physical(self._curl(u))))

    def linearize(self, u):
        self.base = self._physical(u), self._physical(self._curl(u))

    def linear(self, v):
        p, q = self._physical(v), self._physical(self._curl(v))
        return self._spectral(self._cross(p, self.base[1]) + self._cross(self.base[0], q))

    # ---- the implicit solve

    def _helmholtz(self, lam):
        """[k, ny, ny - 2]: from -g_n, n <= N - 2, the solution of (1/Re) (D^2 - lam) f = -g with
        f(+-1) = 0; and the two columns of the wall values."""
        ny, re = self.ny, self.c["re"]
        eye = torch.eye(ny, dtype=torch.float64)
        a = ((self.D @ self.D)[None] - lam[:, None, None] * eye) / re
        n = torch.arange(ny, dtype=torch.float64)
        a[:, ny - 2] = 1.0
        a[:, ny - 1] = (-1.0) ** n
        return torch.linalg.inv(a)

    def _operators(self):
        ny, re = self.ny, self.c["re"]
        n1, nm = ny, ny - 2
        hx, hz = self.nx // 2, self.nz // 2
        k2 = (self.kx[:hx, None] ** 2 + self.kz[None, :hz] ** 2).reshape(-1)
        h = self._helmholtz(k2 + re * self.inv_dt)
        self.Sp = -h[:, :, :nm]           # u_perp, and u and w of the mean mode
        self.wall = h[0, :, nm:]
        # (U, v, p) with U = i u_par: a real system per mode, which falls into two by parity
        d2 = self.D @ self.D
        self.SU = torch.zeros(len(k2), n1, 2 * nm, dtype=torch.float64)
        self.Sv = torch.zeros(len(k2), n1, 2 * nm, dtype=torch.float64)
        one = torch.ones(n1, dtype=torch.float64)
        for e in (0, 1):
            ie, io = torch.arange(e, n1, 2), torch.arange(1 - e, n1, 2)
            re_, ro_ = ie[ie < nm], io[io < nm]
            ne, no = len(ie), len(io)
            size = 2 * ne + no
            k = torch.sqrt(k2[1:])
            a = torch.zeros(len(k), size, size, dtype=torch.float64)
            he = ((d2[ie][:, ie])[None] - (k * k + re * self.inv_dt)[:, None, None]
                  * torch.eye(ne, dtype=torch.float64)) / re
            ho = ((d2[io][:, io])[None] - (k * k + re * self.inv_dt)[:, None, None]
                  * torch.eye(no, dtype=torch.float64)) / re
            r = 0
            a[:, r:r + len(re_), :ne] = he[:, :len(re_)]
            for q in range(len(re_)):
                a[:, r + q, ne + no + q] = k
            r += len(re_)
            a[:, r:r + len(ro_), ne:ne + no] = ho[:, :len(ro_)]
            a[:, r:r + len(ro_), ne + no:] = -self.D[io[:len(ro_)]][:, ie]
            r += len(ro_)
            a[:, r, :ne] = one[:ne]
            a[:, r + 1, ne:ne + no] = one[:no]
            r += 2
            a[:, r:, :ne] = k[:, None, None] * torch.eye(ne, dtype=torch.float64)
            a[:, r:, ne:ne + no] = self.D[ie][:, io]
            rhs = torch.zeros(size, len(re_) + len(ro_), dtype=torch.float64)
            rhs[:len(re_) + len(ro_)] = -torch.eye(len(re_) + len(ro_), dtype=torch.float64)
            x = torch.linalg.solve(a, rhs.expand(len(k), -1, -1))
            cols = torch.cat([re_, nm + ro_])
            sub = torch.zeros(len(k), n1, 2 * nm, dtype=torch.float64)
            sub[:, ie[:, None], cols[None, :]] = x[:, :ne]
            self.SU[1:] += sub
            sub = torch.zeros(len(k), n1, 2 * nm, dtype=torch.float64)
            sub[:, io[:, None], cols[None, :]] = x[:, ne:ne + no]
            self.Sv[1:] += sub

    def _apply(self, m, a):
        """m [hx, hz, r, c] on a [B, nx', hz, c] for the modes m_x >= 0 and m_x < 0 alike."""
        b = a.permute(1, 2, 3, 0).reshape(-1, a.shape[3], a.shape[0])
        y = torch.complex(torch.matmul(m, b.real.contiguous()), torch.matmul(m, b.imag.contiguous()))
        return y.reshape(a.shape[1], a.shape[2], m.shape[1], a.shape[0]).permute(3, 0, 1, 2)

    def solve(self, g, walls):
        """S(g) of [B, 3, nx, nzh, ny]."""
        hx, hz, nm = self.nx // 2, self.nz // 2, self.ny - 2
        out = torch.zeros_like(g)
        per = self.SU.reshape(hx, hz, self.ny, 2 * nm), self.Sv.reshape(hx, hz, self.ny, 2 * nm), \
            self.Sp.reshape(hx, hz, self.ny, nm)
        for rows, modes in ((slice(0, hx), torch.arange(hx)),
                            (slice(hx + 1, self.nx), torch.arange(hx - 1, 0, -1))):
            kx, kz = self.kx[rows][:, None, None], self.kz[:hz][None, :, None]
            k = torch.sqrt(kx * kx + kz * kz)
            k = torch.where(k == 0, torch.ones(()).double(), k)
            f = g[:, :, rows, :hz, :nm]
            par = (kx * f[:, 0] + kz * f[:, 2]) / k
            perp = (kz * f[:, 0] - kx * f[:, 2]) / k
            both = torch.cat([1j * par, f[:, 1]], dim=-1)
            su, sv, sp = (m[modes].reshape(-1, *m.shape[2:]) for m in per)
            upar = -1j * self._apply(su, both)
            uperp = self._apply(sp, perp)
            out[:, 0, rows, :hz] = (kx * upar + kz * uperp) / k
            out[:, 1, rows, :hz] = self._apply(sv, both)
            out[:, 2, rows, :hz] = (kz * upar - kx * uperp) / k
        return self._mean(out, g, walls)

    def _mean(self, out, g, walls):
        nm = self.ny - 2
        sp = self.Sp[0]
        for comp in (0, 1, 2):
            f = g[:, comp, 0, 0, :nm]
            v = torch.complex(f.real @ sp.T, f.imag @ sp.T) if comp != 1 else torch.zeros_like(g[:, 0, 0, 0])
            if walls and comp == 0:
                v = v + (self.wall @ torch.tensor([1.0, -1.0], dtype=torch.float64))
            out[:, comp, 0, 0] = v
        return out

    def _advected_operators(self):
        """Factors of the dense tau systems with the laminar advection."""
        ny, re = self.ny, self.c["re"]
        nm, hz = ny - 2, self.nz // 2
        self.Sp = -self._helmholtz(torch.tensor([re * self.inv_dt], dtype=torch.float64))[:, :, :nm]
        self.wall = self._helmholtz(torch.tensor([re * self.inv_dt], dtype=torch.float64))[0][:, nm:]
        d2 = self.D @ self.D
        y = torch.zeros(ny, ny, dtype=torch.float64)
        y[1, 0] = 1.0
        for n in range(1, ny):
            y[n - 1, n] += 0.5
            if n + 1 < ny:
                y[n + 1, n] += 0.5
        self.Y = y
        modes = [(i, j) for i in range(self.nx) for j in range(hz) if (i, j) != (0, 0) and i != self.nx // 2]
        self.modes = torch.tensor(modes)
        kx, kz = self.kx[self.modes[:, 0]], self.kz[self.modes[:, 1]]
        a = torch.zeros(len(modes), 4 * ny, 4 * ny, dtype=torch.complex128)
        h = (d2[None] - (kx * kx + kz * kz + re * self.inv_dt)[:, None, None] * torch.eye(ny, dtype=torch.float64)) / re
        h = h - 1j * kx[:, None, None] * y
        eye = torch.eye(ny, dtype=torch.float64)[:nm]
        r = 0
        for comp in range(3):
            a[:, r:r + nm, comp * ny:(comp + 1) * ny] = h[:, :nm]
            if comp == 0:
                a[:, r:r + nm, ny:2 * ny] -= eye
                a[:, r:r + nm, 3 * ny:] = -1j * kx[:, None, None] * eye
            elif comp == 1:
                a[:, r:r + nm, 3 * ny:] = -self.D[:nm].to(a.dtype)
            else:
                a[:, r:r + nm, 3 * ny:] = -1j * kz[:, None, None] * eye
            r += nm
        sign = (-1.0) ** torch.arange(ny, dtype=torch.float64)
        for comp in range(3):
            a[:, r, comp * ny:(comp + 1) * ny] = 1.0
            a[:, r + 1, comp * ny:(comp + 1) * ny] = sign.to(a.dtype)
            r += 2
        one = torch.eye(ny, dtype=torch.float64)
        a[:, r:, :ny] = 1j * kx[:, None, None] * one
        a[:, r:, ny:2 * ny] = self.D.to(a.dtype)
        a[:, r:, 2 * ny:3 * ny] = 1j * kz[:, None, None] * one
        self.A = a

    def _advected(self, g, x):
        """(I - dt (L + M))^{-1}: from g and the state x, homogeneous walls."""
        ny, nm = self.ny, self.ny - 2
        g = g + 1j * self.kx[:, None, None] * self._y(self.Y, x)
        g[:, 0] = g[:, 0] + x[:, 1]
        i, j = self.modes[:, 0], self.modes[:, 1]
        f = g[0, :, i, j, :nm].permute(1, 0, 2).reshape(len(i), 3 * nm)
        b = torch.zeros(len(i), 4 * ny, dtype=torch.complex128)
        b[:, :3 * nm] = -f
        z = torch.linalg.solve(self.A, b)[:, :3 * ny].reshape(len(i), 3, ny)
        out = torch.zeros_like(g)
        out[0, :, i, j] = z.permute(1, 0, 2)
        return self._mean(out, g, False)

    # ---- the step and its Jacobian

    def phi(self, u):
        return self.solve(u * self.inv_dt + self.nonlinear(u), True)

    def jvp(self, v):
        g = v * self.inv_dt + self.linear(v)
        return self._advected(g, v) if self.advect else self.solve(g, False)


def _unpack(x, order, shape):
    nx = shape[-3]
    real = torch.zeros(*x.shape[:-1], 2 * int(np.prod(shape)), dtype=torch.float64)
    real = real.index_copy(-1, order, x)
    a = torch.view_as_complex(real.reshape(*x.shape[:-1], *shape, 2))
    mirror = torch.zeros_like(a)
    mirror[..., nx // 2 + 1:, 0, :] = a[..., 1:nx // 2, 0, :].flip(-2).conj()
    return a + mirror


def _pack(a, order, lead=0):
    flat = torch.view_as_real(a.resolve_conj().contiguous()).reshape(*a.shape[:lead], -1)
    return flat.index_select(-1, order)


def exact(case, seed):
    c = case
    if c["kind"] == "newton":
        return None
    f = _fields(c, seed)
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    shape = (3, nx, nz // 2 + 1, ny)
    u = f["u"]
    ref = _Reference(c, advect=c["kind"] == "advect")
    if c["kind"] == "phi":
        return ref.phi(u[None])[0]
    if c["kind"] == "batch":
        return torch.cat([ref.phi(u[i:i + 1]) for i in range(len(u))])
    if c["kind"] == "steps":
        tau = c["dt"]
        if c["scheme"] == 0:
            x = u[None]
            for _ in range(c["steps"]):
                x = ref.phi(x)
            return ((x - u[None]) / (c["steps"] * tau))[0]
        prev, x, before = u[None], u[None], None
        for _ in range(c["steps"]):
            now = ref.nonlinear(x)
            before = now if before is None else before
            g = (4 * x - prev) / 3 / tau + 2 * now - before
            prev, x, before = x, ref.solve(g, True), now
        return ((x - u[None]) / (c["steps"] * 1.5 * tau))[0]
    if c["kind"] in ("jvp", "advect"):
        ref.linearize(u[None])
        v = f["v"][None]
        return _hermitian((ref.jvp(v) - v) / c["dt"])[0]
    order = _packed_order(c)
    if c["kind"] == "columns":
        ref.linearize(u[None])
        n = len(order)
        first = int(seed) * 7919 % max(1, n - c["count"])
        out = torch.zeros(c["count"], n, dtype=torch.float64)
        for a in range(0, c["count"], 32):
            b = min(a + 32, c["count"])
            e = torch.zeros(b - a, n, dtype=torch.float64)
            e[torch.arange(b - a), torch.arange(first + a, first + b)] = 1.0
            v = _unpack(e, order, shape)
            out[a:b] = _pack((ref.jvp(v) - v) / c["dt"], order, 1)
        return out
    # the transposed Jacobian of Phi in the packed product, by torch's own reverse mode
    ref.linearize(u[None])
    x = torch.zeros(len(order), dtype=torch.float64, requires_grad=True)
    y = _pack(ref.jvp(_unpack(x, order, shape)[None])[0], order)
    (gx,) = torch.autograd.grad(y, x, _pack(f["v"], order))
    if c["kind"] == "vjp":
        return _unpack(gx, order, shape)
    return {"y": _pack(ref.phi(u[None])[0], order), "gx": gx}
