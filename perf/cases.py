"""Work that users have this library do, as cases that can be timed and checked.

Every case goes through the public entry points of the Python binding
(`Solver.apply`, `Solver.lanczos_sqrt`) on particles resident in HBM.  Boxes,
densities, heights and forces follow the workloads of this repository: a
sedimented monolayer of driven rollers, a two-layer suspension, uniform
particles; bottom wall and slit channel; float64 and mixed precision; torques
by the spectral curl or by the kernel derivative, or none.

`exact` evaluates the same discrete operator in plain float64 torch with its
own arithmetic: scatter and gather over an 8 x 8 window, torch's FFTs, a
Chebyshev transform by matrix product and one tridiagonal elimination per
parity for all wavenumbers at once.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2210_01837_amd import Solver

BETA_M, BETA_D = 1.327 * 6, 2.216 * 6      # width 6, torques and forces
BETA_4 = 1.87 * 4                          # width 4, forces only
H_SERVE = 1.0 / 1.731                      # spacing at which R_h = 1
R_LAYER = 150.0 / 128.8                    # two-layer box: R_h in cells


def _case(**kw):
    c = dict(kind="apply", geometry="bw", precision="mixed", n=0, nx=0, ny=0,
             nz=32, h=H_SERVE, H=12.0, w=6, beta_m=BETA_M, beta_d=BETA_D,
             heights="monolayer", zlo=0.0, zhi=0.0, unit=1.0, forces="roller",
             torques=True, route="curl", slip0=0.0, slipH=0.0)
    c.update(kw)
    return c


def _forces_only(**kw):
    return _case(**{**dict(h=1.0, H=9.1 * R_LAYER, nz=19, w=4, beta_m=BETA_4,
                           beta_d=BETA_4, heights="bimodal", unit=R_LAYER,
                           forces="gravity", torques=False), **kw})


def listed():
    return [
        # the smallest call: a handful of particles in float64 (a check run, a
        # self mobility); launches and latency count
        _case(name="bw64_fp64", precision="fp64", n=64, nx=48, ny=48,
              h=32.0 / 48, H=8.0, heights="uniform", zlo=1.5, zhi=5.0,
              forces="normal"),
        # the smallest request of a serving stream
        _case(name="serve_bw1k", n=1031, nx=90, ny=90),
        # an ordinary request of that stream between two walls
        _case(name="serve_sc17k", geometry="sc", n=17389, nx=360, ny=360),
        # a float64 channel of uniform particles on a fine Chebyshev grid
        _case(name="sc4096_fp64", geometry="sc", precision="fp64", n=4096,
              nx=192, ny=192, nz=48, h=128.0 / 192, H=10.0, heights="uniform",
              zlo=1.2, zhi=8.8, forces="normal"),
        # a rectangular channel with partial slip on odd grid sizes
        _case(name="sc52k_slip", geometry="sc", n=52361, nx=756, ny=442, nz=27,
              slip0=0.1, slipH=0.05),
        # an ordinary monolayer, as a time step of a simulation computes it
        _case(name="bw131k", n=131072, nx=768, ny=768, h=512.0 / 768),
        # the same in float64, the reference a user compares with
        _case(name="bw131k_fp64", precision="fp64", n=131072, nx=768, ny=768,
              h=512.0 / 768),
        # torques through the kernel derivative
        _case(name="bw300k_derivative", n=300007, nx=1176, ny=1176,
              h=512.0 / 768, route="derivative"),
        # the largest monolayers
        _case(name="bw1m", n=1048576, nx=2176, ny=2176, h=1448.0 / 2176),
        _case(name="sc1m", geometry="sc", n=1048576, nx=2176, ny=2176,
              h=1448.0 / 2176),
        # a forces-only suspension at width 4
        _forces_only(name="layer663k", n=663552, nx=2700, ny=2700),
        # Brownian displacements of a smaller one, to three digits
        _forces_only(name="lanczos18k", kind="lanczos", n=18432, nx=450, ny=450),
    ]


def _even_size(rng, x, primes):
    """An even grid size near x with prime factors among `primes`."""
    c = max(24, int(round(x)))
    near = []
    for v in range(max(24, int(0.93 * c)), int(1.07 * c) + 3):
        m = v
        for p in primes:
            while m % p == 0:
                m //= p
        if m == 1 and v % 2 == 0:
            near.append(v)
    return rng.choice(near or [c + c % 2 if not c % 32 else 32 * (c // 32 + 1)])


def draw(rng):
    log = lambda a, b: int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))   # noqa: E731
    primes = rng.choice([(2, 3, 5, 7), (2, 3, 5, 7), (2, 3, 5, 7, 11, 13, 17)])
    family = rng.choice(["monolayer", "monolayer", "monolayer", "serve", "serve",
                         "serve", "fp64", "fp64", "fine", "derivative", "slip",
                         "layer", "layer", "lanczos"])
    geometry = rng.choice(["bw", "sc"])
    if family in ("layer", "lanczos"):
        n = log(512, 524288) if family == "layer" else log(512, 32768)
        side = math.sqrt(n / 2048.0) * 150.0
        return _forces_only(kind="apply" if family == "layer" else "lanczos",
                            n=n, nx=_even_size(rng, side, primes),
                            ny=_even_size(rng, side, primes))
    h = 2.0 / 3.0 if family == "monolayer" else H_SERVE
    kw = dict(geometry=geometry, h=h, nz=rng.choice([32, 32, 31, 28, 25]))
    if family == "fp64":
        n, kw["precision"] = log(64, 98304), "fp64"
    elif family == "fine":
        n = log(256, 16384)
        kw.update(precision=rng.choice(["fp64", "mixed"]), nz=rng.choice([40, 48]),
                  geometry="sc", heights="uniform", zlo=1.2, zhi=10.8,
                  forces="normal")
    else:
        n = log(64 if family == "monolayer" else 1024, 524288)
        if family == "derivative":
            kw["route"] = "derivative"
        if family == "slip":
            n = min(n, 262144)
            kw.update(geometry="sc", slip0=rng.choice([0.05, 0.1, 0.3]),
                      slipH=rng.choice([0.0, 0.05, 0.2]))
    side = math.sqrt(n / rng.uniform(0.4, 0.5)) / h
    aspect = rng.choice([1.0, 1.0, 1.3])
    return _case(n=n, nx=_even_size(rng, side * aspect, primes),
                 ny=_even_size(rng, side / aspect, primes), **kw)


# --- inputs -----------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _inputs(c, seed):
    """(pos, F, T) or (pos, W) in the solver's type."""
    g = torch.Generator(device=_device()).manual_seed(int(seed))
    n = c["n"]
    kw = dict(generator=g, device=_device(), dtype=torch.float64)
    uni = lambda: torch.rand(n, **kw)     # noqa: E731
    nrm = lambda *s: torch.randn(*s, **kw)   # noqa: E731
    x, y = uni() * (c["nx"] * c["h"]), uni() * (c["ny"] * c["h"])
    if c["heights"] == "uniform":
        z = c["zlo"] + (c["zhi"] - c["zlo"]) * uni()
    else:
        z = 1.1 - 0.3 * torch.log1p(-uni())
        if c["heights"] == "bimodal":
            high = (3.3 + 0.3 * nrm(n)).clamp(2.4, 5.0)
            z = c["unit"] * torch.where(uni() < 0.5, z, high)
    if c["forces"] == "normal":
        F, T = nrm(n, 3), nrm(n, 3)
    else:
        F, T = 0.1 * nrm(n, 3), 0.1 * nrm(n, 3)
        F[:, 2] -= 1.0
        T[:, 1] += 1.0
    if c["kind"] == "lanczos":
        F = nrm(n, 3)
    t = torch.float64 if c["precision"] == "fp64" else torch.float32
    pos = torch.stack([x, y, z], 1).to(t)
    # rounding may carry a coordinate past the last float below the period; it
    # is wrapped by the library like any other
    return pos, F.to(t), (T.to(t) if c["torques"] else None)


def prepare(case, seed):
    pos, F, T = _inputs(case, seed)
    c = case
    solver = Solver(c["geometry"], c["nx"] * c["h"], c["ny"] * c["h"], c["H"],
                    c["nx"], c["ny"], c["nz"], w=c["w"], beta_m=c["beta_m"],
                    beta_d=c["beta_d"], precision=c["precision"],
                    max_particles=c["n"], slip0=c["slip0"], slipH=c["slipH"],
                    torque_route=c["route"])
    return {"kind": c["kind"], "solver": solver, "pos": pos, "F": F, "T": T}


def run(state):
    s = state["solver"]
    if state["kind"] == "lanczos":
        g, iterations, _ = s.lanczos_sqrt(state["pos"], state["F"], max_iter=32,
                                          tol=1e-3)
        return {"g": g, "iterations": iterations}
    U, Om = s.apply(state["pos"], state["F"], state["T"],
                    want_omega=state["T"] is not None)
    return {"U": U} if Om is None else {"U": U, "Omega": Om}


def work(case):
    """Particle arrays once, and the arithmetic of the method: spread and
    interpolation, transforms of the planes that particles reach, column
    solves."""
    c = case
    size = 8 if c["precision"] == "fp64" else 4
    n, nz, nxy = c["n"], c["nz"], c["nx"] * c["ny"]
    alpha = 0.5 * c["w"] * c["h"]
    zc = 0.5 * c["H"] * (1 + np.cos(np.pi * np.arange(nz) / (nz - 1)))
    top = {"uniform": c["zhi"], "bimodal": 5.0 * c["unit"],
           "monolayer": 1.1 + 0.3 * math.log(n)}[c["heights"]]
    planes = int(np.sum(zc <= top + alpha))
    mid = 0.5 * (1.1 * c["unit"] + top)
    window = int(np.sum(np.abs(zc - mid) <= alpha))
    both = 2 if c["torques"] else 1
    ch = 3 * both if c["route"] == "curl" else 3
    per_window = (c["w"] + 1) ** 2 * window * 6.0 * both
    fft = ch * planes * 2.5 * nxy * math.log2(nxy)
    columns = 0.5 * nxy * 2 * (2 * ch * 2.5 * nz * math.log2(nz) + 4 * 14.0 * nz)
    flops = 2 * n * per_window + 2 * fft + columns
    arrays = 3 * n * size * (2 + 1 + 2 * (both - 1))
    if c["kind"] == "lanczos":
        # the iterations to three digits; positions, W and g once
        return {"bytes": 9.0 * n * size, "flops": 12.0 * flops}
    return {"bytes": float(arrays), "flops": float(flops)}


# --- the operator in float64 ------------------------------------------------

class _Exact:
    def __init__(self, c):
        self.c = c
        self.dev = _device()
        self.h, self.H, self.nz = c["h"] * c["nx"] / c["nx"], c["H"], c["nz"]
        self.alpha = 0.5 * c["w"] * self.h
        self.Lx, self.Ly = c["nx"] * c["h"], c["ny"] * c["h"]
        n = np.arange(self.nz)
        T = np.cos(np.pi * np.outer(n, n) / (self.nz - 1))
        M = T * (2.0 / (self.nz - 1))
        M[[0, -1], :] *= 0.5
        M[:, [0, -1]] *= 0.5
        integral = np.where(n % 2 == 0, 2.0 / (1.0 - n.astype(float) ** 2 + (n == 1)), 0.0)
        self.zc = self._t(0.5 * self.H * (1.0 + np.cos(np.pi * n / (self.nz - 1))))
        self.quad = self._t(self.h ** 2 * 0.5 * self.H * (M.T @ integral))
        self.to_coef, self.to_node = self._t(M), self._t(T)
        x, wq = np.polynomial.legendre.leggauss(200)
        th = 0.5 * np.pi * x
        self.norm = {b: float(self.alpha * 0.5 * np.pi * np.sum(
            wq * np.exp(b * (np.cos(th) - 1.0)) * np.cos(th)))
            for b in (c["beta_m"], c["beta_d"])}
        # truncation of the dipole kernel's derivative
        roots = np.roots([c["beta_d"], 0.0, -c["beta_d"], 1.0])
        s = sorted(r.real for r in roots if abs(r.imag) < 1e-12 and 0 < r.real < 1)
        self.tstar = self.alpha * math.sqrt(1.0 - s[0] ** 2) if s else self.alpha

    def _t(self, a):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64,
                               device=self.dev)

    def _phi(self, t, beta):
        r = t / self.alpha
        s = ((1.0 - r) * (1.0 + r)).clamp(min=0.0).sqrt()
        return torch.where(t.abs() <= self.alpha,
                           torch.exp(beta * (s - 1.0)) / self.norm[beta], 0.0)

    def _dphi(self, t, beta):
        keep = t.abs() <= self.tstar
        r = torch.where(keep, t / self.alpha, 0.0)
        s = ((1.0 - r) * (1.0 + r)).sqrt()
        return torch.where(keep, self._phi(t, beta) * beta * (-r / self.alpha) / s, 0.0)

    def _fold(self, f, z, beta):
        zc, z = self.zc[None, :], z[:, None]
        v = f(zc - z, beta) - f(zc + z, beta)
        if self.c["geometry"] == "sc":
            v = v - f(zc - (2.0 * self.H - z), beta)
        return v

    def set_particles(self, pos):
        """Window indices and separable weights: terms 0 (monopole), and 1
        (dipole) or 1..3 (dipole derivative along x, along y, none)."""
        c, p = self.c, pos.double()
        bm, bd = c["beta_m"], c["beta_d"]

        def axis(x, L, N):
            u = torch.remainder(x, L) / self.h
            a = torch.floor(u)[:, None] + torch.arange(-3, 5, device=self.dev)
            t = (a - u[:, None]) * self.h
            return a.long() % N, self._phi(t, bm), self._phi(t, bd), self._dphi(t, bd)

        self.ia, xm, xd, xe = axis(p[:, 0], self.Lx, c["nx"])
        self.ib, ym, yd, ye = axis(p[:, 1], self.Ly, c["ny"])
        zm, zd, ze = (self._fold(f, p[:, 2], b) for f, b in
                      ((self._phi, bm), (self._phi, bd), (self._dphi, bd)))
        reach = torch.nonzero(((zm != 0) | (ze != 0)).any(0)).flatten()
        self.lo, self.hi = int(reach[0]), int(reach[-1]) + 1
        zm, zd, ze = (v[:, self.lo:self.hi] for v in (zm, zd, ze))
        self.P = self.hi - self.lo
        if not c["torques"]:
            self.terms = [(xm, ym)]
        elif c["route"] == "curl":
            self.terms = [(xm, ym), (xd, yd)]
        else:
            self.terms = [(xm, ym), (xe, yd), (xd, ye), (xd, yd)]
        self.zm, self.zd, self.ze = zm, zd, ze

    def _chunks(self, n, size=131072):
        return [slice(i, min(n, i + size)) for i in range(0, n, size)]

    def _values(self, sl, F, T):
        """Per term, the (m, channels, planes) values it adds to the grid."""
        outer = lambda v, z: v[:, :, None] * z[:, None, :]   # noqa: E731
        zm, zd, ze = self.zm[sl], self.zd[sl], self.ze[sl]
        vals = [outer(F[sl], zm)]
        if len(self.terms) == 2:
            vals.append(outer(T[sl], zd))
        elif len(self.terms) == 4:
            t = 0.5 * T[sl]
            o = torch.zeros_like(t[:, 0])
            vals.append(outer(torch.stack([o, -t[:, 2], t[:, 1]], 1), zd))
            vals.append(outer(torch.stack([t[:, 2], o, -t[:, 0]], 1), zd))
            vals.append(outer(torch.stack([-t[:, 1], t[:, 0], o], 1), ze))
        return vals

    def spread(self, F, T):
        c, P = self.c, self.P
        ch = 6 if len(self.terms) == 2 else 3
        grid = torch.zeros(c["ny"] * c["nx"], ch * P, dtype=torch.float64, device=self.dev)
        for sl in self._chunks(F.shape[0]):
            vals = self._values(sl, F, T)
            for i in range(8):
                for j in range(8):
                    parts = [(wx[sl, i] * wy[sl, j])[:, None, None] * v
                             for (wx, wy), v in zip(self.terms, vals)]
                    v = torch.cat(parts, 1) if ch == 6 else sum(parts)
                    grid.index_add_(0, self.ib[sl, j] * c["nx"] + self.ia[sl, i],
                                    v.reshape(v.shape[0], -1))
        return grid

    def _gather(self, grid, sl, term, cols):
        wx, wy = term
        acc = 0.0
        for i in range(8):
            for j in range(8):
                rows = grid[self.ib[sl, j] * self.c["nx"] + self.ia[sl, i]][:, cols]
                acc = acc + (wx[sl, i] * wy[sl, j])[:, None] * rows
        return acc.reshape(acc.shape[0], 3, self.P)

    def interp(self, grid):
        q = self.quad[self.lo:self.hi]
        U, Om = [], []
        front, back = slice(0, 3 * self.P), slice(3 * self.P, 6 * self.P)
        for sl in self._chunks(self.ia.shape[0]):
            U.append((self._gather(grid, sl, self.terms[0], front)
                      * (self.zm[sl] * q)[:, None, :]).sum(-1))
            zd, ze = self.zd[sl] * q, self.ze[sl] * q
            if len(self.terms) == 2:
                Om.append((self._gather(grid, sl, self.terms[1], back)
                           * zd[:, None, :]).sum(-1))
            elif len(self.terms) == 4:
                gx, gy = (self._gather(grid, sl, t, front) * zd[:, None, :]
                          for t in self.terms[1:3])
                gz = self._gather(grid, sl, self.terms[3], front) * ze[:, None, :]
                gx, gy, gz = gx.sum(-1), gy.sum(-1), gz.sum(-1)
                Om.append(0.5 * torch.stack([gz[:, 1] - gy[:, 2], gx[:, 2] - gz[:, 0],
                                             gy[:, 0] - gx[:, 1]], 1))
        return torch.cat(U), (torch.cat(Om) if Om else None)

    # Chebyshev series as (nz, columns) tensors
    def _deriv(self, a):
        b = [None] * self.nz
        zero = torch.zeros_like(a[0])
        b[-1] = zero
        for n in range(self.nz - 1, 0, -1):
            v = (b[n + 1] if n + 1 < self.nz else zero) + 2.0 * n * a[n]
            b[n - 1] = 0.5 * v if n == 1 else v
        return torch.stack(b) * (2.0 / self.H)

    def _b2(self, r):
        """Rows m >= 2 of the double antiderivative (rows 0, 1 zero)."""
        out = torch.zeros_like(r)
        for m in range(2, self.nz):
            v = (2.0 if m == 2 else 1.0) / (4.0 * m * (m - 1)) * r[m - 2]
            v = v - r[m] / (2.0 * (m * m - 1.0))
            if m + 2 < self.nz:
                v = v + r[m + 2] / (4.0 * m * (m + 1))
            out[m] = v
        return out

    def _operator(self, kappa):
        """Elimination of y - kappa^2 B^2 y = b, rows m >= 2, from the last
        row: y_m = al_m y_{m-2} + be_m."""
        al, inv, up = {}, {}, {}
        k2 = kappa * kappa
        for m in range(self.nz - 1, 1, -1):
            up[m] = k2 / (4.0 * m * (m + 1)) if m + 2 < self.nz else torch.zeros_like(k2)
            d = 1.0 + k2 / (2.0 * (m * m - 1.0))
            if m + 2 < self.nz:
                d = d - up[m] * al[m + 2]
            inv[m] = 1.0 / d
            al[m] = (2.0 if m == 2 else 1.0) * k2 / (4.0 * m * (m - 1)) * inv[m]
        return kappa, al, inv, up

    def _robin(self, op, r, gH, g0):
        kappa, al, inv, up = op
        b = (0.25 * self.H ** 2) * self._b2(r)
        be, y = {}, [None] * self.nz
        for m in range(self.nz - 1, 1, -1):
            be[m] = inv[m] * (b[m] + (up[m] * be[m + 2] if m + 2 < self.nz else 0.0))
        for p in (0, 1):
            # boundary rows: sum over the parity of (m^2 + kappa) y_m
            Pm, Qm = torch.ones_like(kappa), torch.zeros_like(b[0])
            E, S = p * p + kappa, torch.zeros_like(b[0])
            chain = []
            for m in range(p + 2, self.nz, 2):
                Pm, Qm = al[m] * Pm, al[m] * Qm + be[m]
                chain.append((m, Pm, Qm))
                E = E + (m * m + kappa) * Pm
                S = S + (m * m + kappa) * Qm
            g = 0.25 * self.H * (gH - g0 if p == 0 else gH + g0)
            y[p] = (g - S) / E
            for m, Pm, Qm in chain:
                y[m] = Pm * y[p] + Qm
        return torch.stack(y)

    def _sums(self, a):
        """Values and z-derivatives at z = H and z = 0."""
        n = torch.arange(self.nz, device=self.dev, dtype=torch.float64)[:, None]
        alt, s = 1.0 - 2.0 * (n % 2), 2.0 / self.H
        return (a.sum(0), (alt * a).sum(0), s * (n * n * a).sum(0),
                s * (-alt * n * n * a).sum(0))

    @staticmethod
    def _small_solve(A, b):
        """Gaussian elimination with partial pivoting, real A[row][col] and
        complex b as (rows, columns...) tensors."""
        n = A.shape[0]
        rows = torch.arange(n, device=A.device)[:, None]
        for c in range(n):
            piv = A[c:, c].abs().argmax(0) + c
            order = torch.where(rows == c, piv, torch.where(rows == piv, c, rows))
            A = A.gather(0, order[:, None, :].expand_as(A))
            b = b.gather(0, order)
            if c + 1 < n:
                f = A[c + 1:, c] / A[c, c]
                A = torch.cat([A[:c + 1], A[c + 1:] - f[:, None] * A[c]])
                b = torch.cat([b[:c + 1], b[c + 1:] - f * b[c]])
        x = [None] * n
        for c in range(n - 1, -1, -1):
            s = b[c]
            for k in range(c + 1, n):
                s = s - A[c, k] * x[k]
            x[c] = s / A[c, c]
        return x

    def _correction(self, kx, ky, k, u, v, w):
        """Node values of the flow that restores the wall conditions."""
        H, l0, lH = self.H, self.c["slip0"], self.c["slipH"]
        uH, u0, uHd, u0d = self._sums(u)
        vH, v0, vHd, v0d = self._sums(v)
        wH, w0, _, _ = self._sums(w)
        u0, v0, w0 = -u0 + l0 * u0d, -v0 + l0 * v0d, -w0
        z = self.zc[:, None]
        em = torch.exp(-k * z)
        if self.c["geometry"] == "bw":
            B = k * w0 - 1j * (kx * u0 + ky * v0)
            return (-(1j * kx / k) * B * z * em + u0 * em,
                    -(1j * ky / k) * B * z * em + v0 * em, B * z * em + w0 * em)
        uH, vH, wH = -uH - lH * uHd, -vH - lH * vHd, -wH
        # along k, i times the velocity is real like w; across k on its own
        cx, cy = kx / k, ky / k
        a0, t0 = 1j * (cx * u0 + cy * v0), cx * v0 - cy * u0
        aH, tH = 1j * (cx * uH + cy * vH), cx * vH - cy * uH
        E, o, z0 = torch.exp(-k * H), torch.ones_like(k), torch.zeros_like(k)
        hh, kl0, klH = 0.5 * H, k * l0, k * lH
        A = torch.stack([torch.stack(r) for r in (
            (-0.5 * l0 * o, 0.5 * l0 * E, 1 + kl0, (1 - kl0) * E, z0, z0),
            (z0, z0, z0, z0, o, E),
            (hh * E * (1 + lH / H - klH), -hh * (1 + lH / H + klH), E * (1 - klH), 1 + klH, z0, z0),
            (hh * E, hh * o, z0, z0, E, o),
            (0.5 * o, 0.5 * E, k, k * E, -k, k * E),
            (0.5 * E, 0.5 * o, k * E, k, -k * E, k))])
        zc = torch.zeros_like(w0)
        C0, D0, iC, iD, Cz, Dz = self._small_solve(A, torch.stack([a0, w0, aH, wH, zc, zc]))
        det = (1 + kl0) * (1 + klH) - (1 - kl0) * (1 - klH) * E * E
        CT = ((1 + klH) * t0 - (1 - kl0) * E * tH) / det
        DT = ((1 + kl0) * tH - E * (1 - klH) * t0) / det
        ep = torch.exp(k * (z - H))
        along = -1j * (0.5 * z * (C0 * em - D0 * ep) + iC * em + iD * ep)
        across = CT * em + DT * ep
        return (cx * along - cy * across, cy * along + cx * across,
                0.5 * z * (C0 * em + D0 * ep) + Cz * em + Dz * ep)

    def _zero_mode(self, f):
        """y'' = -f for the mean flow: one column, by dense elimination."""
        n, H = np.arange(self.nz, dtype=float), self.H
        s, alt = 2.0 / H, (-1.0) ** np.arange(self.nz)
        A = np.eye(self.nz)
        b = 0.25 * H * H * self._b2(-f).cpu().numpy()
        A[1], b[1] = alt + self.c["slip0"] * s * alt * n ** 2, 0.0
        A[0] = n ** 2 if self.c["geometry"] == "bw" else 1.0 + self.c["slipH"] * s * n ** 2
        b[0] = 0.0
        return torch.as_tensor(np.linalg.solve(A, b), device=self.dev)

    def columns(self, spec, kx, ky):
        """(channels, planes, columns) spectra of the densities -> of the
        velocity (and half vorticity), in place of them."""
        def transform(M, a):
            r = torch.view_as_real(a.contiguous()).reshape(a.shape[0], -1)
            return torch.view_as_complex((M @ r).reshape(M.shape[0], a.shape[1], 2))
        coef = self.to_coef[:, self.lo:self.hi].contiguous()
        f = [transform(coef, s) for s in spec]
        if len(f) == 6:
            gx, gy, gz = f[3:]
            f = [f[0] + 0.5 * (1j * ky * gz - self._deriv(gy)),
                 f[1] + 0.5 * (self._deriv(gx) - 1j * kx * gz),
                 f[2] + 0.5 * (1j * kx * gy - 1j * ky * gx)]
        zero = (kx == 0) & (ky == 0)
        k = torch.where(zero, 1.0, (kx * kx + ky * ky).sqrt())
        op = self._operator(0.5 * k * self.H)
        none = torch.zeros_like(f[0][0])
        p = self._robin(op, 1j * kx * f[0] + 1j * ky * f[1] + self._deriv(f[2]), none, none)
        pH, p0, _, _ = self._sums(p)
        u = self._robin(op, 1j * kx * p - f[0], -0.5j * kx / k * pH, 0.5j * kx / k * p0)
        v = self._robin(op, 1j * ky * p - f[1], -0.5j * ky / k * pH, 0.5j * ky / k * p0)
        w = self._robin(op, self._deriv(p) - f[2], 0.5 * pH, 0.5 * p0)
        cu = self._correction(kx, ky, k, u, v, w)
        u, v, w = (a + transform(self.to_coef, b) for a, b in zip((u, v, w), cu))
        for j in torch.nonzero(zero).flatten().tolist():
            u[:, j], v[:, j], w[:, j] = self._zero_mode(f[0][:, j]), self._zero_mode(f[1][:, j]), 0.0
        out = [u, v, w]
        if spec.shape[0] == 6:
            out += [0.5 * (1j * ky * w - self._deriv(v)), 0.5 * (self._deriv(u) - 1j * kx * w),
                    0.5 * (1j * kx * v - 1j * ky * u)]
        node = self.to_node[self.lo:self.hi].contiguous()
        nyq = (kx == math.pi / self.h) | (ky.abs() == math.pi / self.h)
        for s, a in zip(spec, out):
            s.copy_(torch.where(nyq, 0.0, transform(node, a)))

    def apply(self, F, T):
        c = self.c
        nx, ny, nk = c["nx"], c["ny"], c["nx"] // 2 + 1
        grid = self.spread(F.double(), None if T is None else T.double())
        ch = grid.shape[1] // self.P
        spec = torch.empty(ch * self.P, ny, nk, dtype=torch.complex128, device=self.dev)
        for j in range(ch * self.P):
            spec[j] = torch.fft.rfft2(grid[:, j].reshape(ny, nx))
        f64 = dict(device=self.dev, dtype=torch.float64)
        kx = torch.arange(nk, **f64) * (2.0 * math.pi / self.Lx)
        ky = torch.fft.fftfreq(ny, d=1.0 / ny, **f64) * (2.0 * math.pi / self.Ly)
        kx[-1] = math.pi / self.h          # Nyquist modes, dropped below
        ky[ny // 2] = math.pi / self.h
        kx, ky = kx.repeat(ny), ky.repeat_interleave(nk)
        flat = spec.view(ch, self.P, ny * nk)
        for sl in self._chunks(ny * nk, 262144):
            part = flat[:, :, sl].clone()
            self.columns(part, kx[sl], ky[sl])
            flat[:, :, sl] = part
        for j in range(ch * self.P):
            grid[:, j] = torch.fft.irfft2(spec[j], s=(ny, nx)).reshape(-1)
        return self.interp(grid)


def _sqrt_e1(alpha, beta, norm):
    T = np.diag(alpha) + np.diag(beta[:len(alpha) - 1], 1) + np.diag(beta[:len(alpha) - 1], -1)
    lam, Q = np.linalg.eigh(T)
    return norm * (Q @ (np.sqrt(np.maximum(lam, 0.0)) * Q[0]))


def exact(case, seed):
    pos, F, T = _inputs(case, seed)
    op = _Exact(case)
    op.set_particles(pos)
    if case["kind"] == "apply":
        U, Om = op.apply(F, T)
        return {"U": U} if Om is None else {"U": U, "Omega": Om}
    # Lanczos process, stopped at the same relative change
    W = F.double().reshape(-1)
    norm = float(W.norm())
    V, alpha, beta, last = [W / norm], [], [], None
    for j in range(32):
        r = op.apply(V[j].reshape(-1, 3), None)[0].reshape(-1)
        basis = torch.stack(V)
        first = basis @ r
        alpha.append(float(first[j]))
        r = r - basis.T @ first
        r = r - basis.T @ (basis @ r)
        beta.append(float(r.norm()))
        y = _sqrt_e1(alpha, beta, norm)
        if last is not None and (np.linalg.norm(y - np.append(last, 0.0))
                                 < 1e-3 * np.linalg.norm(last)):
            break
        last = y
        V.append(r / beta[-1])
    g = torch.stack(V[:len(y)]).T @ torch.as_tensor(y, device=op.dev)
    return {"g": g.reshape(-1, 3), "iterations": None}
