"""Cases by which the speed of the library is judged: what a program that uses it has it do.

A DG fast spectral solver calls the collision operator on every quadrature point of its mesh, so the ordinary call is
a batch of velocity-space functions: one point (a homogeneous relaxation, a probe), the 30 points of a small 1-D
mesh, hundreds to thousands on production meshes.  The grids are 16^3 to 48^3 points, FP32 with the FP64 fix or plain
FP64.  Besides the operator itself (with its conservation projection) a program calls the 1-D driver's time step, the
weak form in the paper's SVD factors and, for gradients, the vector-Jacobian product.  Each listed case is one of
these at a size of the repository's own workloads or its tests; `draw` spreads the same calls over their ranges.

`exact` is the plain Fourier spectral formula in 64 bits with torch.fft.
"""
import functools
import math
import os

import numpy as np
import torch

import paper_1809_10186_amd as qc

DEV = "cuda:0"


def _case(name, kind, N, L, Nr, M, omega, items, fp64=False, alpha=1.0, svd_tol=0.0, T=(0.5, 2.0), umax=0.5,
          tune=False, K=3, follows=True):
    c = dict(kind=kind, N=N, L=L, Nr=Nr, M=M, omega=omega, items=items, fp64=fp64, alpha=alpha, svd_tol=svd_tol,
             T_lo=T[0], T_hi=T[1], umax=umax, tune=tune, K=K, follows=follows)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one point, Maxwell molecules on 16^3, B = 1/(4 pi): one right-hand side of the space-homogeneous BKW
        # relaxation (thousands of these in sequence: latency is all that counts)
        _case("relax16_fp64_1", "eval", 16, 8.0, 8, 6, 1.0, 1, fp64=True, follows=False),
        # one point on the production grid: a probe, a debugger, a point solver that calls the operator per cell
        _case("point32_fp32_1", "eval", 32, 6.0, 16, 12, 0.81, 1),
        # one SSP-RK2 step of the 1-D driver, Fourier heat transfer: 10 elements of order 2, 24^3, M = 6, Maxwell
        # molecules, both precisions
        _case("fourier24_fp32_step", "dg1d", 24, 5.09, 12, 6, 1.0, 10),
        _case("fourier24_fp64_step", "dg1d", 24, 5.09, 12, 6, 1.0, 10, fp64=True),
        # the 1D DG batch: 64 elements x 3 Gauss points, 32^3, gain table truncated at 1e-8, autotuned, both precisions
        _case("dg1d32_fp32_192", "eval", 32, 6.0, 16, 12, 0.81, 192, svd_tol=1e-8, tune=True),
        _case("dg1d32_fp64_192", "eval", 32, 6.0, 16, 12, 0.81, 192, fp64=True, svd_tol=1e-8, tune=True),
        # a 2D DG batch (16 x 16 elements of 2 x 2 points), 24^3
        _case("dg2d24_fp32_1024", "eval", 24, 6.0, 12, 12, 0.74, 1024, tune=True),
        # the hot 48^3 grid of the three-grid shock batch, gain table truncated at 1e-6
        _case("shock48_fp32_307", "eval", 48, 9.0, 24, 12, 0.81, 307, svd_tol=1e-6, T=(2.5, 3.5), umax=2.3),
        # gradients of a loss through the projected operator, df and domega: a mini-batch in FP32, a ragged small
        # one in FP64 (a gradient check, an adjoint solve)
        _case("vjp32_fp32_256", "vjp", 32, 6.0, 16, 12, 0.81, 256),
        _case("vjp32_fp64_37", "vjp", 32, 6.0, 16, 12, 0.81, 37, fp64=True),
        # VSS scattering (alpha = 1.5) in FP64 on an odd number of points
        _case("vss32_fp64_45", "eval", 32, 6.0, 16, 12, 0.81, 45, fp64=True, alpha=1.5),
        # the weak form in the paper's SVD factors (bilinear Q): 16 elements of order 2, 6 terms each
        _case("dgsvd32_fp32_16", "dgsvd", 32, 6.0, 16, 12, 0.81, 16),
    ]


def _evals(c):
    """Operator evaluations of one pass (items, nodes and stages taken together)."""
    per = {"eval": 1, "vjp": 1, "dg1d": 2 * c["K"], "dgsvd": c["K"] * (c["K"] - 1)}[c["kind"]]
    return c["items"] * per


def _flops_per_eval(c):
    n = c["N"] ** 3
    fft = 5.0 * n * math.log2(n)
    per_term = {"eval": fft + 23.0 * n, "dg1d": fft + 23.0 * n, "vjp": 2 * fft + 30.0 * n, "dgsvd": 2 * fft + 30.0 * n}
    t = per_term[c["kind"]] + (fft if c["alpha"] != 1.0 else 0.0)
    return c["Nr"] * c["M"] * t + (c["Nr"] + 4) * fft


def draw(rng):
    """One call of the same kinds: a grid, a rule, a precision and a batch (spread over its logarithm)."""
    kind = rng.choice(["eval", "eval", "eval", "eval", "vjp", "vjp", "dg1d", "dgsvd"])
    N = rng.choice({"eval": [8, 12, 16, 24, 32, 32, 48], "vjp": [16, 24, 32, 32], "dg1d": [16, 24, 32],
                    "dgsvd": [16, 24, 32]}[kind])
    fp64 = rng.random() < 0.4
    M = rng.choice([6, 12, 12, 16])
    Nr = rng.randint(4, 16) if N <= 32 else rng.randint(12, 24)
    alpha = round(rng.uniform(1.2, 1.9), 2) if kind == "eval" and N <= 32 and rng.random() < 0.25 else 1.0
    omega = round(rng.uniform(0.5, 1.0), 3)
    # operator evaluations within half of the largest listed case's arithmetic; the paths that keep their volumes
    # in memory take about three times as long per operation
    c = _case(None, kind, N, 6.0 if N <= 32 else 9.0, Nr, M, omega, 1, fp64, alpha,
              T=(0.5, 2.0) if N <= 32 else (2.5, 3.5), umax=0.5 if N <= 32 else 2.0, K=rng.choice([2, 3]))
    slow = 3.0 if fp64 or N > 32 or kind == "dgsvd" else 1.0
    most = max(1, min(4096, int(1.0e12 / (slow * _flops_per_eval(c) * _evals(c)))))
    c["items"] = max(1, int(math.exp(rng.uniform(0.0, math.log(most + 0.99)))))
    if kind == "dg1d":
        c["items"] = max(2, min(c["items"], 64))
    if kind == "dgsvd":
        c["items"] = min(c["items"], 128)
    return c


def work(c):
    n = c["N"] ** 3
    ev = _evals(c)
    tables = n * c["Nr"] * (8 if c["fp64"] else 4) * (c["M"] / 2.0 if c["alpha"] != 1.0 else 1.0) + 8.0 * n
    state = {"eval": 2 * ev, "vjp": 3 * ev, "dg1d": 2 * c["items"] * c["K"], "dgsvd": 2 * c["items"] * c["K"]}[c["kind"]]
    return {"bytes": 8.0 * n * state + tables, "flops": ev * _flops_per_eval(c)}


# --------------------------------------------------------------------------
# inputs

def _sphere(M):
    a = np.loadtxt(os.path.join("workloads", "sphere", f"half_M{M}.txt"))
    return np.ascontiguousarray(a[:, :3]), np.ascontiguousarray(a[:, 3])


def _nodes(N, L):
    return (torch.arange(N, dtype=torch.float64, device=DEV) + 0.5) * (2.0 * L / N) - L


def _gauss(N, L, n, u, T):
    """Maxwellians n (pi T)^{-3/2} exp(-|c - u|^2 / T): [B, N, N, N]."""
    c = _nodes(N, L)
    e = [torch.exp(-(c[None] - u[:, d, None]) ** 2 / T[:, None]) for d in range(3)]
    a = n / (math.pi * T) ** 1.5
    return (a[:, None, None, None] * e[0][:, :, None, None]) * e[1][:, None, :, None] * e[2][:, None, None, :]


def _mixtures(c, B, seed):
    """Two-Maxwellian states with 1% positive noise, as near walls and shocks."""
    r = np.random.default_rng(seed)
    f = None
    for _ in range(2):
        d = r.normal(size=(B, 3))
        d *= (c["umax"] * r.random(B) ** (1.0 / 3.0) / np.linalg.norm(d, axis=1))[:, None]
        t = [torch.from_numpy(x).to(DEV) for x in (r.uniform(0.5, 1.5, B), d, r.uniform(c["T_lo"], c["T_hi"], B))]
        g = _gauss(c["N"], c["L"], *t)
        f = g if f is None else f.add_(g)
    gen = torch.Generator(DEV)
    gen.manual_seed(seed)
    f.mul_(1.0 + 0.01 * torch.rand(f.shape, generator=gen, dtype=torch.float64, device=DEV))
    return f


def _cotangent(f, seed):
    gen = torch.Generator(DEV)
    gen.manual_seed(seed + 7919)
    return f * torch.randn(f.shape, generator=gen, dtype=torch.float64, device=DEV)


def _faces(E):
    """Elements refined towards both walls (ratio 1.23 for ten), on [0, 1]."""
    h = 1.23 ** np.minimum(np.arange(E), np.arange(E)[::-1]).clip(max=8)
    return np.concatenate([[0.0], np.cumsum(h / h.sum())])


def _lagrange(K):
    """Gauss nodes and weights, phi_l(-1), phi_l(+1), and phi_l'(xi_q)."""
    x, w = np.polynomial.legendre.leggauss(K)
    P = np.polynomial.polynomial
    co = [P.polyfromroots(np.delete(x, l)) for l in range(K)]
    co = [a / P.polyval(x[l], a) for l, a in enumerate(co)]
    at = lambda y: np.array([P.polyval(y, a) for a in co])  # noqa: E731
    return x, w, at(-1.0), at(1.0), np.array([P.polyval(x, P.polyder(a)) for a in co]), at


def _svd_factors(K):
    """The paper's factors of the triple tensor: rows of T1, T2 and the weights W (singular values above rounding)."""
    at = _lagrange(K)[-1]
    xq, wq = np.polynomial.legendre.leggauss(3 * K)
    ph = at(xq)
    H = np.einsum("q,mq,aq,bq->mab", wq, ph, ph, ph)
    T1, T2, W = [], [], []
    for m in range(K):
        U, s, V = np.linalg.svd(H[m])
        for i in range(K):
            if s[i] > 1e-12 * s[0]:
                T1.append(U[:, i])
                T2.append(V[i])
                col = np.zeros(K)
                col[m] = s[i]
                W.append(col)
    return [torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (np.array(T1), np.array(T2), np.array(W).T)]


DT = 0.002
INV_KN = (math.pi / 2.0) / 1.582
T_WALL = (263.0 / 273.0, 283.0 / 273.0)


def _dg1d_state(c, seed):
    """Maxwellians near equilibrium on every node of the mesh."""
    r = np.random.default_rng(seed)
    B = c["items"] * c["K"]
    t = [torch.from_numpy(x).to(DEV) for x in (r.uniform(0.9, 1.1, B), 0.05 * r.normal(size=(B, 3)),
                                               r.uniform(0.95, 1.05, B))]
    n = c["N"]
    return _gauss(n, c["L"], *t).reshape(c["items"], c["K"], n, n, n)


def _plan(c):
    svd = dict(svd_rank=0, svd_tol=c["svd_tol"]) if c["svd_tol"] else {}
    return qc.Plan(c["N"], c["L"], c["Nr"], sphere=_sphere(c["M"]), omega=c["omega"], alpha=c["alpha"],
                   prefactor=None if c["follows"] else 1.0 / (4.0 * math.pi),
                   precision=qc.QCOLL_FP64 if c["fp64"] else qc.QCOLL_FP32, **svd)


def prepare(c, seed):
    torch.cuda.set_device(0)
    s = {"kind": c["kind"], "plan": _plan(c)}
    if c["kind"] == "dg1d":
        s["F0"] = _dg1d_state(c, seed)
        s["F"] = torch.empty_like(s["F0"])
        s["dg"] = qc.Dg1d(s["plan"], _faces(c["items"]), c["K"] - 1, INV_KN, qc.Bc("wall", T=T_WALL[0]),
                          qc.Bc("wall", T=T_WALL[1]))
    elif c["kind"] == "dgsvd":
        n = c["N"]
        s["F"] = _mixtures(c, c["items"] * c["K"], seed).reshape(c["items"], c["K"], n, n, n)
        s["C"] = torch.empty_like(s["F"])
        s["factors"] = _svd_factors(c["K"])
    else:
        s["f"] = _mixtures(c, c["items"], seed)
        s["out"] = torch.empty_like(s["f"])
        if c["kind"] == "vjp":
            s["g"] = _cotangent(s["f"], seed)
            s["dw"] = torch.empty(c["items"], dtype=torch.float64, device=DEV)
        elif c["tune"]:
            s["plan"].autotune(s["f"], s["out"])
    return s


def run(s):
    plan, kind = s["plan"], s["kind"]
    if kind == "eval":
        plan.eval(s["f"], s["out"])
        return plan.conserve(s["out"])
    if kind == "vjp":
        df, dw = plan.vjp(s["f"], s["g"], df=s["out"], domega=s["dw"], through_conserve=True, want_domega=True)
        return {"df": df, "domega": dw}
    if kind == "dg1d":
        s["F"].copy_(s["F0"])       # the state before the step is kept: a step can be rejected
        return s["dg"].step(s["F"], DT, rk=2)
    T1, T2, W = s["factors"]
    return plan.dg_collide_svd(s["F"], T1, T2, W, conserve=True, out=s["C"])


# --------------------------------------------------------------------------
# the same in 64 bits, without the library

@functools.lru_cache(maxsize=None)
def _gauss_jacobi(n, A):
    """Nodes and weights for the weight (1 - t)^A on [-1, 1], from the matrix of the three-term recurrence."""
    i = np.arange(n, dtype=float)
    d = -A * A / ((2 * i + A) * (2 * i + A + 2))
    d[0] = -A / (A + 2)
    j = i[1:]
    e = 4 * j * (j + A) * j * (j + A) / ((2 * j + A) ** 2 * (2 * j + A + 1) * (2 * j + A - 1))
    t, v = np.linalg.eigh(np.diag(d) + np.diag(np.sqrt(e), 1) + np.diag(np.sqrt(e), -1))
    return t, v[0] ** 2 * 2.0 ** (A + 1) / (A + 1)


class _Exact:
    def __init__(self, c):
        self.c = c
        N, L, om, al = c["N"], c["L"], c["omega"], c["alpha"]
        self.N, self.L, self.M = N, L, c["M"]
        R = 4.0 * L / (3.0 + math.sqrt(2.0))
        x, w = np.polynomial.legendre.leggauss(c["Nr"])
        self.rho, self.wr = 0.5 * R * (x + 1.0), 0.5 * R * w
        self.pts, self.wq = _sphere(self.M)
        self.b = al / (2.0 ** (2.0 - om + al) * math.gamma(2.5 - om) * math.pi) if c["follows"] else 0.25 / math.pi
        k = torch.arange(N, dtype=torch.float64, device=DEV)
        self.k = torch.where(k < N // 2, k, k - N)
        k1, k2, k3 = torch.meshgrid(self.k, self.k, self.k, indexing="ij")
        self.kv = torch.stack([k1, k2, k3], -1)
        ka = self.kv.square().sum(-1).sqrt()
        self.vss = al != 1.0
        wsum = float(self.wq.sum())
        if self.vss:
            self.alpha = None
            self.lam_p = torch.zeros((c["Nr"], N, N, N), dtype=torch.float64, device=DEV)
            for p in range(c["Nr"]):
                for q in range(self.M):
                    self.lam_p[p] += 2.0 * self.wr[p] * self.wq[q] * self._F_vss(2.0, p, q)
        else:
            F = lambda ks, r: 4.0 * math.pi * self.b * r ** (4.0 - 2.0 * om) * torch.sinc(r * ks / (2.0 * L))  # noqa: E731
            self.alpha = torch.stack([2.0 * w * F(ka, r) for r, w in zip(self.rho, self.wr)])
            self.lam_p = torch.stack([2.0 * wsum * w * F(2.0 * ka, r) for r, w in zip(self.rho, self.wr)])
            if c["svd_tol"]:
                A = self.alpha.reshape(c["Nr"], -1).cpu().numpy()
                U, s, V = np.linalg.svd(A, full_matrices=False)
                m = int((s > c["svd_tol"] * s[0]).sum())
                self.alpha = torch.from_numpy(((U[:, :m] * s[:m]) @ V[:m]).reshape(self.alpha.shape)).to(DEV)
        self.lam = self.lam_p.sum(0)
        g = _nodes(N, L)
        c1, c2, c3 = torch.meshgrid(g, g, g, indexing="ij")
        self.cv = torch.stack([c1, c2, c3])
        self.inv = torch.stack([torch.ones_like(c1), c1, c2, c3, self.cv.square().sum(0)]).reshape(5, -1)
        self.ginv = torch.linalg.inv((self.inv @ self.inv.T).cpu()).to(DEV)

    def _F_vss(self, mult, p, q):
        """F(mult k, rho_p, sigma_q) for the symmetrised VSS kernel; indices at -N/2 averaged over their signs."""
        N, al, rho = self.N, self.c["alpha"], self.rho[p]
        sig = torch.from_numpy(self.pts[q]).to(DEV)

        def F(kv):
            kab = kv.square().sum(-1).sqrt()
            a = math.pi * rho * kab / (2.0 * self.L)
            mu = torch.where(kab > 0, (kv @ sig) / kab.clamp(min=1e-30), torch.ones_like(kab)).clamp(-1.0, 1.0)
            nu = (1.0 - mu * mu).sqrt()
            n = int(1.25 * math.pi * rho * mult * N * 0.87 / (2.0 * self.L)) + 48
            t, wt = (torch.from_numpy(x).to(DEV) for x in _gauss_jacobi(n, al - 1.0))
            s = (1.0 - t * t).clamp(min=0.0).sqrt()
            z = (a * nu)[..., None] * s
            m = 20 + int(0.55 * float(z.max()))     # J0(z) = mean of cos(z cos phi): the midpoint rule, to rounding
            j0 = 0.0
            for i in range(m):
                j0 = j0 + torch.cos(z * math.cos(math.pi * (i + 0.5) / m)) / m
            out = (torch.cos((a * mu)[..., None] * t) * j0) @ wt
            return 2.0 * math.pi * self.b * rho ** (4.0 - 2.0 * self.c["omega"]) * out

        out = F(mult * self.kv)
        nyq = self.kv.abs() == N // 2
        at = nyq.any(-1)
        ks, ns = self.kv[at], nyq[at]
        sg = 1.0 - 2.0 * torch.tensor(list(np.ndindex(2, 2, 2)), dtype=torch.float64, device=DEV)
        out[at] = F(mult * ks * torch.where(ns, sg[:, None, :], torch.ones_like(ks))).mean(0)
        return out

    def _beta(self, p, q):
        b = []
        for d in range(3):
            th = math.pi * self.k * (0.5 * self.rho[p] * self.pts[q, d]) / self.L
            z = torch.complex(torch.cos(th), torch.sin(th))
            z[self.N // 2] = torch.cos(th[self.N // 2])
            b.append(z)
        return b[0][:, None, None] * b[1][None, :, None] * b[2][None, None, :]

    @staticmethod
    def _fft(x):
        return torch.fft.fftn(x, dim=(-3, -2, -1))

    @staticmethod
    def _ifft(x):
        return torch.fft.ifftn(x, dim=(-3, -2, -1))

    def _chunks(self, B):
        n = max(1, int(1.5e8 / self.N ** 3))
        return [slice(i, min(B, i + n)) for i in range(0, B, n)]

    def project(self, Q):
        q = Q.reshape(-1, self.N ** 3)
        return (q - ((q @ self.inv.T) @ self.ginv) @ self.inv).reshape(Q.shape)

    def Q(self, f, g=None):
        """Q(f, f), or the bilinear Q(f, g)."""
        out = torch.empty_like(f)
        for s in self._chunks(f.shape[0]):
            X = self._fft(f[s])
            Y = X if g is None else self._fft(g[s])
            Qh = torch.zeros_like(X)
            for p in range(len(self.rho)):
                A = 0.0
                for q in range(self.M):
                    bt = self._beta(p, q)
                    # t1 + i t2 = ifft[(beta + i conj(beta)) X], both real
                    m = bt + 1j * bt.conj()
                    u = self._ifft(m * X)
                    if g is None:
                        t = u.real * u.imag
                    else:
                        v = self._ifft(m * Y)
                        t = 0.5 * (u.real * v.imag + u.imag * v.real)
                    if self.vss:
                        Qh += 2.0 * self.wr[p] * self.wq[q] * self._F_vss(1.0, p, q) * self._fft(t)
                    else:
                        A = A + self.wq[q] * t
                if not self.vss:
                    Qh += self.alpha[p] * self._fft(A)
            out[s] = self._ifft(Qh).real - f[s] * self._ifft(self.lam * Y).real
        return out

    def vjp(self, f, g):
        g = self.project(g)
        df, dw = torch.empty_like(f), torch.empty(f.shape[0], dtype=torch.float64, device=DEV)
        dlog = math.log(2.0) + float(torch.digamma(torch.tensor(2.5 - self.c["omega"], dtype=torch.float64)))
        for s in self._chunks(f.shape[0]):
            X, G = self._fft(f[s]), self._fft(g[s])
            acc = torch.zeros_like(X)
            w = 0.0
            for p in range(len(self.rho)):
                h = self._ifft(self.alpha[p] * G).real
                gain = 0.0
                for q in range(self.M):
                    bt = self._beta(p, q)
                    u = self._ifft((bt + 1j * bt.conj()) * X)
                    t1, t2 = u.real, u.imag
                    # the transpose of a shift is the opposite shift
                    acc += self.wq[q] * (bt.conj() * self._fft(h * t2) + bt * self._fft(h * t1))
                    gain = gain + self.wq[q] * (h * t1 * t2).sum((1, 2, 3))
                loss = (f[s] * g[s] * self._ifft(self.lam_p[p] * X).real).sum((1, 2, 3))
                w = w + (dlog - 2.0 * math.log(self.rho[p])) * (gain - loss)
            df[s] = self._ifft(acc).real - g[s] * self._ifft(self.lam * X).real \
                - self._ifft(self.lam * self._fft(f[s] * g[s])).real
            dw[s] = w
        return df, dw

    def rhs(self, F, faces):
        """The semi-discrete right-hand side of the 1-D driver, collocated collision term, diffuse walls."""
        E, K = F.shape[:2]
        _, w, pl, pr, dphi, _ = _lagrange(K)
        as_t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
        S, Lm, Rm = as_t(w[None, :] * dphi), as_t(pl), as_t(pr)
        J = as_t(0.5 * np.diff(faces))
        cx = self.cv[0]
        fR, fL = torch.einsum("l,el...->e...", Rm, F), torch.einsum("l,el...->e...", Lm, F)

        def wall(trace, sign, T):
            fw, cn = torch.exp(-self.cv.square().sum(0) / T), cx * sign
            return -(cn * trace)[cn >= 0].sum() / (cn * fw)[cn < 0].sum() * fw

        ext_R = torch.cat([fL[1:], wall(fR[-1], 1.0, T_WALL[1])[None]])
        ext_L = torch.cat([wall(fL[0], -1.0, T_WALL[0])[None], fR[:-1]])
        sR, sL = torch.where(cx >= 0, fR, ext_R), torch.where(cx > 0, ext_L, fL)
        out = torch.einsum("ml,el...->em...", S, F) * cx
        out -= Rm[None, :, None, None, None] * (cx * sR)[:, None]
        out += Lm[None, :, None, None, None] * (cx * sL)[:, None]
        out /= J[:, None, None, None, None] * as_t(w)[None, :, None, None, None]
        return out + INV_KN * self.project(self.Q(F.flatten(0, 1))).reshape(F.shape)


def exact(c, seed):
    torch.cuda.set_device(0)
    e = _Exact(c)
    if c["kind"] == "eval":
        return e.project(e.Q(_mixtures(c, c["items"], seed)))
    if c["kind"] == "vjp":
        f = _mixtures(c, c["items"], seed)
        df, dw = e.vjp(f, _cotangent(f, seed))
        return {"df": df, "domega": dw}
    if c["kind"] == "dg1d":
        F, faces = _dg1d_state(c, seed), _faces(c["items"])
        v = F + DT * e.rhs(F, faces)
        return 0.5 * F + 0.5 * v + 0.5 * DT * e.rhs(v, faces)
    n = c["N"]
    F = _mixtures(c, c["items"] * c["K"], seed).reshape(c["items"], c["K"], n, n, n)
    T1, T2, W = _svd_factors(c["K"])
    a, b = (torch.einsum("rk,ek...->er...", T, F).flatten(0, 1).contiguous() for T in (T1, T2))
    q = e.project(e.Q(a, b)).reshape(c["items"], T1.shape[0], n, n, n)
    return torch.einsum("kr,er...->ek...", W, q)
