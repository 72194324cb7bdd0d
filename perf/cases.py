"""The library's workloads, measured through its public entry points.

Each case is one pass of something that a lattice program does with a
``wcl.Lattice``: operator applications on its own fields (one vector or a
batch, FP64 / FP32 / FP16 tiers, D and its adjoint, the even/odd and Schwarz
steps), taking in a new gauge field, solves of D x = b with the solvers the
library offers, and the gradient of a solve.  Links are near-unit SU(3)
matrices, exp(i 0.3 H) with H Hermitian, traceless and complex Gaussian;
sources are complex Gaussian or the 12 spin-colour point sources.  ``exact``
holds the same mathematics in plain torch at 64 bits.
"""
import itertools
import math

import torch

from paper_1612_06556_amd import autograd, wcl

CSW = 1.0
LINK = {(64, 0): 144, (32, 0): 72, (16, 0): 36, (32, 1): 48, (16, 1): 24}
CLOV = {64: 576, 32: 288, 16: 144}
OPS = {"hop": wcl.OP_HOP, "clover_inv": wcl.OP_CLOVER_INV, "schur": wcl.OP_SCHUR, "ras": wcl.OP_RAS}


def listed():
    return [
        # the smallest call: one vector on 8^4, launches and latency
        _case("d_fp64_8", "apply", (8, 8, 8, 8), prec=64, dagger=False, nrhs=1, two_row=0),
        # the residual of an adjoint system on the paper's lattice
        _case("ddag_fp64_24", "apply", (24, 24, 24, 32), prec=64, dagger=True, nrhs=1, two_row=0),
        # the 12 spin-colour vectors of a propagator in the half-precision tier
        _case("d_fp16_12src_16", "apply", (16, 16, 16, 32), prec=16, dagger=False, nrhs=12, two_row=1),
        # one single-precision application on the largest lattice of the benchmark
        _case("d_fp32_32", "apply", (32, 32, 32, 64), prec=32, dagger=False, nrhs=1, two_row=0),
        # the even/odd operator on a lattice whose extents 4 does not divide
        _case("schur_fp32_ragged", "op", (12, 6, 10, 14), op="schur", prec=32, nrhs=2, two_row=0),
        # one Schwarz application, the benchmark's preconditioner
        _case("ras_fp32_24", "op", (24, 24, 24, 32), op="ras", prec=32, nrhs=1, two_row=1),
        # a new gauge field (a Monte Carlo step): links, clover term, then one D
        _case("gauge_24", "gauge", (24, 24, 24, 32), two_row=1),
        # the benchmark's solve: FP64 outer, FP32 two-row inner with Schwarz
        _case("solve_ras_24", "solve", (24, 24, 24, 32), kappa=0.126, solver="ras_fp32", nrhs=1, two_row=1),
        # a 12-source propagator with the fastest inner tier (FP16 links and vectors)
        _case("solve_12src_fp16_16", "solve", (16, 16, 16, 32), kappa=0.125, solver="noras_fp16", nrhs=12, two_row=1),
        # the plain FP64 even/odd solver on the differentiation workload's lattice
        _case("solve_fp64_eo_16", "solve", (16, 16, 16, 32), kappa=0.125, solver="fp64_eo", nrhs=1, two_row=0),
        # link and kappa gradients from two solutions
        _case("grad_16", "grad", (16, 16, 16, 32), kappa=0.125),
        # one differentiable step on a small lattice: forward solve, adjoint solve, gradients
        _case("train_8", "train", (8, 8, 8, 8), kappa=0.12),
    ]


def _case(name, kind, dims, kappa=0.125, **kw):
    c = {"kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], "kappa": kappa, **kw}
    if name:
        c["name"] = name
    return c


def draw(rng):
    """A case of the listed kinds: even extents from 6 up (half of them lattices
    that 4 does not divide), volumes spread over their logarithm."""
    kind = rng.choice(["apply", "apply", "op", "op", "gauge", "solve", "solve", "grad", "train"])
    top = {"apply": 32 ** 3 * 64, "op": 24 ** 3 * 32, "gauge": 24 ** 3 * 32, "solve": 16 ** 3 * 32,
           "grad": 16 ** 3 * 32, "train": 8 ** 3 * 16}[kind]
    dims = _dims(rng, 8 ** 4, top)
    V = math.prod(dims)
    two_row = rng.randrange(2)
    if kind == "apply":
        most = max(1, min(12, 2 ** 21 // V))
        return _case(None, kind, dims, prec=rng.choice([64, 32, 16]), dagger=rng.random() < 0.4,
                     nrhs=rng.choice([n for n in (1, 1, 2, 3, 5, 12) if n <= most]), two_row=two_row)
    if kind == "op":
        op = rng.choice(list(OPS))
        prec = rng.choice([32, 16] if op == "ras" else [64, 32, 16])
        return _case(None, kind, dims, op=op, prec=prec, nrhs=rng.choice([1, 1, 2, 3] if V < 10 ** 5 else [1]),
                     two_row=two_row)
    if kind == "gauge":
        return _case(None, kind, dims, two_row=two_row)
    if kind == "solve":
        solver = rng.choice(["ras_fp32", "noras_fp32", "noras_fp16", "fp64_eo", "fp64_full"])
        return _case(None, kind, dims, kappa=rng.choice([0.115, 0.12, 0.125]), solver=solver,
                     nrhs=rng.choice([1, 1, 3, 12] if V < 40000 else [1, 1, 2]), two_row=two_row)
    return _case(None, kind, dims, kappa=rng.choice([0.11, 0.115, 0.12]))


def _dims(rng, low, top):
    want = math.exp(rng.uniform(math.log(low), math.log(top)))
    step, ragged = (2, True) if rng.random() < 0.5 else (4, False)
    while True:
        d = [rng.randrange(8 - (2 if ragged else 0), 37, step) for _ in range(3)]
        t = int(want / math.prod(d) / step + 0.5) * step
        if 6 <= t <= 96 and low // 2 <= math.prod(d) * t <= top and (not ragged or any(x % 4 for x in (*d, t))):
            if ragged or t >= 8:
                return (*d, t)


# --- inputs -------------------------------------------------------------------

def _dims_of(c):
    return c["lx"], c["ly"], c["lz"], c["lt"]


def _links(dims, gen):
    """[V, 4, 3, 3] SU(3) links exp(i 0.3 H), rows re-orthonormalised."""
    n = math.prod(dims) * 4
    out = torch.empty((n, 3, 3), dtype=torch.complex128, device="cuda")
    for s in range(0, n, 1 << 21):
        m = min(1 << 21, n - s)
        a = torch.randn((m, 3, 3), dtype=torch.complex128, device="cuda", generator=gen)
        h = 0.5 * (a + a.mH)
        tr = (h[:, 0, 0] + h[:, 1, 1] + h[:, 2, 2]) / 3.0
        h = 0.3j * (h - tr[:, None, None] * torch.eye(3, dtype=h.dtype, device=h.device))
        e = torch.eye(3, dtype=h.dtype, device=h.device).expand(m, 3, 3)
        for k in range(14, 0, -1):
            e = torch.eye(3, dtype=h.dtype, device=h.device) + _mul(h, e) / k
        r0 = e[:, 0] / torch.linalg.vector_norm(e[:, 0], dim=-1, keepdim=True)
        r1 = e[:, 1] - (r0.conj() * e[:, 1]).sum(-1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
        out[s:s + m] = torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=1)
    return out.view(-1, 4, 3, 3)


def _fields(c, seed):
    """(U, vectors) of a case: what its program has in hand, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dims = _dims_of(c)
    V = math.prod(dims)
    U = _links(dims, gen)

    def spinor(*lead):
        return torch.randn((*lead, V, 4, 3), dtype=torch.complex128, device="cuda", generator=gen)

    n = c.get("nrhs", 1)
    if c["kind"] in ("grad", "train"):
        return U, (spinor(), spinor())
    if c["kind"] == "solve" and n == 12:
        b = torch.zeros((12, V, 4, 3), dtype=torch.complex128, device="cuda")
        site = int(torch.randint(V, (1,), device="cuda", generator=gen))
        for k in range(12):
            b[k, site, k // 3, k % 3] = 1.0
        return U, (b,)
    return U, (spinor(n) if n > 1 else spinor(),)


def _solver_options(c):
    """wcl.Lattice.solve options; the solution is wanted to about 1e-10."""
    return {
        "ras_fp32": dict(tol=1e-11, inner_tol=0.1),
        "noras_fp32": dict(tol=1e-11, inner_tol=0.1, use_ras=0),
        "noras_fp16": dict(tol=1e-11, inner_tol=0.1, use_ras=0, inner_prec=16, inner_vec_prec=16),
        "fp64_eo": dict(tol=1e-11, outer=wcl.OUTER_PLAIN64_EO, max_outer=5000),
        "fp64_full": dict(tol=1e-11, outer=wcl.OUTER_PLAIN64, max_outer=5000),
    }[c["solver"]]


def prepare(c, seed):
    U, vec = _fields(c, seed)
    lat = wcl.Lattice(_dims_of(c), -1)
    lat.set_compression(c.get("two_row", 0))
    lat.set_gauge(U)
    lat.set_params(c["kappa"], CSW)
    st = {"case": c, "lat": lat, "vec": vec}
    if c["kind"] == "train":
        st["U"] = U.requires_grad_(True)
        st["kappa"] = torch.tensor(c["kappa"], dtype=torch.float64, requires_grad=True)
        st["b"] = vec[0].requires_grad_(True)
    elif c["kind"] == "gauge":
        st["U"] = U
    elif c["kind"] == "solve":
        st["opts"] = _solver_options(c)
    return st


def run(st):
    c, lat, vec = st["case"], st["lat"], st["vec"]
    kind = c["kind"]
    if kind == "apply":
        return lat.apply(vec[0], dagger=c["dagger"], prec=c["prec"])
    if kind == "op":
        return lat.apply_op(OPS[c["op"]], vec[0], prec=c["prec"])
    if kind == "gauge":
        lat.set_gauge(st["U"])
        lat.set_params(c["kappa"], CSW)
        return lat.apply(vec[0])
    if kind == "solve":
        return lat.solve(vec[0], **st["opts"])[0]
    if kind == "grad":
        gU, gk = lat.grad(vec[0], vec[1])
        return {"gU": gU, "gkappa": gk}
    x = autograd.solve(st["U"], st["kappa"], st["b"], lat, csw=CSW, tol=1e-11, inner_tol=0.1)
    gU, gk, gb = torch.autograd.grad(x, (st["U"], st["kappa"], st["b"]), vec[1])
    return {"x": x.detach(), "gU": gU, "gkappa": gk, "gb": gb}


def work(c):
    """Bytes: canonical complex128 inputs and outputs and the resident operator
    fields, each once; flops: 1320 per hop site, 504 per clover site, 48 per
    axpy; solves: a representative iteration count of two Schur applications."""
    V, n, p = math.prod(_dims_of(c)), c.get("nrhs", 1), c.get("prec", 64)
    vec = 192.0 * V
    op = V * (4.0 * LINK[(p, c.get("two_row", 0) if p < 64 else 0)] + CLOV[p])
    d_flops = V * 1872.0
    kind = c["kind"]
    if kind == "apply":
        return {"bytes": 2 * n * vec + op, "flops": n * d_flops}
    if kind == "op":
        if c["op"] == "hop":
            return {"bytes": 2 * n * vec + op - V * CLOV[p], "flops": n * V * 1320.0}
        if c["op"] == "clover_inv":
            return {"bytes": 2 * n * vec + V * CLOV[p], "flops": n * V * 504.0}
        if c["op"] == "schur":
            return {"bytes": 1.5 * n * vec + op, "flops": n * d_flops}
        # 4 steps on 6^4 (or 4^4) blocks around 4^4 (or 2^4) cores
        core = 4 if all(d % 4 == 0 for d in _dims_of(c)) else 2
        e = (core + 2) ** 4
        per = 8.0 * (core + 1) / (core + 2) * e * 168 + e * 504 + e / 2 * 240
        return {"bytes": 1.5 * n * vec + op, "flops": n * 4.0 * per * V / core ** 4}
    setup = {"bytes": V * 576.0 * 3, "flops": V * (6 * 4 * 3 * 198 + 2 * 1500.0)}
    if kind == "gauge":
        return {"bytes": setup["bytes"] + 2 * vec, "flops": setup["flops"] + d_flops}
    grad = {"bytes": V * 576.0 * 2 + 2 * vec, "flops": V * (4 * 6 * 9 * 198.0 + 2 * 1320)}
    if kind == "grad":
        return grad
    its = {"ras_fp32": 30, "noras_fp32": 100, "noras_fp16": 90, "fp64_eo": 62, "fp64_full": 125}
    s, reps = (c["solver"], 1) if kind == "solve" else ("noras_fp32", 2)
    it, per = its[s] * n * reps, 2 * V * 1872.0
    if s == "ras_fp32":
        per += 2 * work(dict(c, kind="op", op="ras", prec=32, nrhs=1))["flops"]
    size = {"ras_fp32": 32, "noras_fp32": 32, "noras_fp16": 16, "fp64_eo": 64, "fp64_full": 64}[s]
    out = {"bytes": 2 * n * vec * reps + V * (4.0 * LINK[(size, 0)] + CLOV[size]), "flops": it * per}
    if kind == "train":
        out = {k: out[k] + 2 * setup[k] + grad[k] for k in out}
    return out


# --- the same in plain torch at 64 bits ----------------------------------------
# Fields as [.., Lt, Lz, Ly, Lx, ..]; direction mu (x, y, z, t) rolls axis 3 - mu
# of the site axes.  gamma_k = [[0, -i s_k], [i s_k, 0]], gamma_t = [[0, 1], [1, 0]].

_PAULI = ([[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]])


def _pauli(k):
    return torch.tensor(_PAULI[k], dtype=torch.complex128, device="cuda")


def _upper(mu):
    """G_mu of gamma_mu = [[0, G], [G^dag, 0]]."""
    return -1j * _pauli(mu) if mu < 3 else torch.eye(2, dtype=torch.complex128, device="cuda")


def _mul(a, b):
    return (a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :])


def _spin(m, psi):
    """m (2x2 in spin) on [.., 2, 3]."""
    a, b = psi[..., 0:1, :], psi[..., 1:2, :]
    return torch.cat([m[0, 0] * a + m[0, 1] * b, m[1, 0] * a + m[1, 1] * b], dim=-2)


def _colour(u, h):
    """u (3x3 in colour) on [.., spin, 3]."""
    return sum(u[..., None, :, k] * h[..., k:k + 1] for k in range(3))


class _Wilson:
    """D = T - kappa H from the links, differentiable in U and kappa."""

    def __init__(self, dims, U, kappa):
        Lx, Ly, Lz, Lt = dims
        self.dims, self.kappa = dims, kappa
        self.shape = (Lt, Lz, Ly, Lx)
        self.U = [U.reshape(*self.shape, 4, 3, 3)[..., mu, :, :] for mu in range(4)]
        sign = torch.ones((Lt, 1, 1, 1, 1, 1), dtype=torch.complex128, device="cuda")
        sign[-1] = -1.0
        hop = self.U[:3] + [self.U[3] * sign]
        self.fwd = hop
        self.bwd = [torch.roll(u, 1, 3 - mu).mH for mu, u in enumerate(hop)]
        self.chi = self._clover()

    def _leaves(self, mu, nu):
        a, b = 3 - mu, 3 - nu
        um, un = self.U[mu], self.U[nu]
        unp, ump = torch.roll(un, -1, a), torch.roll(um, -1, b)       # U_nu(x+mu), U_mu(x+nu)
        umm, unm = torch.roll(um, 1, a), torch.roll(un, 1, a)         # at x - mu
        q = _mul(_mul(um, unp), _mul(ump.mH, un.mH))
        q = q + _mul(_mul(un, torch.roll(ump, 1, a).mH), _mul(unm.mH, umm))
        umn, unn = torch.roll(um, 1, b), torch.roll(un, 1, b)         # at x - nu
        q = q + _mul(_mul(umm.mH, torch.roll(unm, 1, b).mH), _mul(torch.roll(umm, 1, b), unn))
        return q + _mul(_mul(unn.mH, umn), _mul(torch.roll(unp, 1, b), um.mH))

    def _clover(self):
        """The two 6x6 blocks of T (spins 0, 1 and spins 2, 3)."""
        eye3 = torch.eye(3, dtype=torch.complex128, device="cuda")
        gam = []
        for mu in range(4):
            g = torch.zeros((4, 4), dtype=torch.complex128, device="cuda")
            g[:2, 2:], g[2:, :2] = _upper(mu), _upper(mu).mH
            gam.append(g)
        out = [0.0, 0.0]
        for mu, nu in itertools.combinations(range(4), 2):
            q = self._leaves(mu, nu)
            f = (q - q.mH) / 8j
            f = f - (f.diagonal(dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None] * eye3
            sig = 0.5j * (gam[mu] @ gam[nu] - gam[nu] @ gam[mu])
            for k in range(2):
                s = sig[2 * k:2 * k + 2, 2 * k:2 * k + 2]
                out[k] = out[k] + (s[:, None, :, None] * f[..., None, :, None, :]).reshape(*self.shape, 6, 6)
        eye6 = torch.eye(6, dtype=torch.complex128, device="cuda")
        return [eye6 - CSW * self.kappa * t for t in out]

    @staticmethod
    def chiral(blocks, psi):
        """Two 6x6 blocks on [.., 4, 3]."""
        v = [psi[..., :2, :].flatten(-2), psi[..., 2:, :].flatten(-2)]
        return torch.cat([sum(t[..., :, k] * x[..., k:k + 1] for k in range(6)).unflatten(-1, (2, 3))
                          for t, x in zip(blocks, v)], dim=-2)

    def hop(self, psi, sign=1):
        """H psi, or with sign -1 the projectors swapped."""
        out = 0.0
        for mu in range(4):
            ax = psi.dim() - 3 - mu
            G = _upper(mu)
            for d, u, s in ((-1, self.fwd[mu], -sign), (1, self.bwd[mu], sign)):
                p = torch.roll(psi, d, ax)
                h = _colour(u, p[..., :2, :] + s * _spin(G, p[..., 2:, :]))
                out = out + torch.cat([h, s * _spin(G.mH, h)], dim=-2)
        return out

    def D(self, psi):
        return self.chiral(self.chi, psi) - self.kappa * self.hop(psi)

    def Ddag(self, psi):
        return self.chiral(self.chi, psi) - self.kappa * self.hop(psi, -1)

    def inv(self):
        return [torch.linalg.inv(t) for t in self.chi]

    def parity(self):
        i = [torch.arange(n, device="cuda") for n in self.shape]
        return ((i[0][:, None, None, None] + i[1][:, None, None] + i[2][:, None] + i[3]) & 1)[..., None, None]

    def solve(self, b, tol=1e-13):
        """BiCGStab on the even/odd system, right-hand sides side by side."""
        even, ti, k2 = self.parity() == 0, self.inv(), self.kappa ** 2

        def schur(v):
            y = torch.where(even, 0.0, self.chiral(ti, self.hop(v)))
            return v - k2 * torch.where(even, self.chiral(ti, self.hop(y)), 0.0)

        def dot(u, v):
            return (u.conj() * v).flatten(-6).sum(-1)[..., None, None, None, None, None, None]

        tb = self.chiral(ti, b)
        bh = torch.where(even, tb + self.kappa * self.chiral(ti, self.hop(torch.where(even, 0.0, tb))), 0.0)
        x, bn = torch.zeros_like(bh), dot(bh, bh).real.clamp_min(1e-300)
        for _ in range(6):
            r = bh - schur(x)
            rt, rho, al, om, v, p = r, 1.0, 1.0, 1.0, torch.zeros_like(r), torch.zeros_like(r)
            rn0 = dot(r, r).real
            for it in range(400):
                if float((dot(r, r).real / bn).max()) < tol ** 2:
                    break
                rho, old = dot(rt, r), rho
                p = r + (rho / old) * (al / om) * (p - om * v)
                v = schur(p)
                al = rho / dot(rt, v)
                s = r - al * v
                t = schur(s)
                om = dot(t, s) / dot(t, t)
                x = x + al * p + om * s
                r = s - om * t
                if bool((dot(r, r).real < 1e-16 * rn0).all()):
                    break
            r = bh - schur(x)
            if float((dot(r, r).real / bn).max()) < tol ** 2:
                break
        return x + torch.where(even, 0.0, tb + self.kappa * self.chiral(ti, self.hop(x)))

    def ras(self, v, iters=4):
        """Minimal residual on each core extended by one site, hops that leave
        it dropped, from zero; the even sites of the core are kept."""
        core = 4 if all(d % 4 == 0 for d in self.dims) else 2
        e = core + 2
        dev = v.device
        nb = [n // core for n in self.shape]
        at = []
        for ax, n in enumerate(self.shape):
            k = (torch.arange(nb[ax], device=dev)[:, None] * core + torch.arange(e, device=dev) - 1) % n
            at.append(k.reshape([nb[a] if a == ax else 1 for a in range(4)] + [e if a == ax else 1 for a in range(4)]))
        idx = 0
        for k, n in zip(at, self.shape):
            idx = idx * n + k
        idx = idx.reshape(-1, e, e, e, e)
        even = (self.parity() == 0).flatten()[idx][..., None, None]
        site = v.reshape(-1, 4, 3)
        U = [u.reshape(-1, 3, 3)[idx] for u in self.fwd]
        ti = [t.reshape(-1, 6, 6)[idx] for t in self.inv()]

        def hop(psi):
            out = torch.zeros_like(psi)
            for mu in range(4):
                ax, G = 4 - mu, _upper(mu)
                lo, hi = (slice(None),) * ax + (slice(0, e - 1),), (slice(None),) * ax + (slice(1, e),)
                u = U[mu][lo]
                for src, dst, w, s in ((hi, lo, u, -1), (lo, hi, u.mH, 1)):
                    p = psi[src]
                    h = _colour(w, p[..., :2, :] + s * _spin(G, p[..., 2:, :]))
                    out[dst] += torch.cat([h, s * _spin(G.mH, h)], dim=-2)
            return out

        r = torch.where(even, site[idx], 0.0)
        z = torch.zeros_like(r)
        for _ in range(iters):
            y = torch.where(even, 0.0, self.chiral(ti, hop(r)))
            q = r - self.kappa ** 2 * torch.where(even, self.chiral(ti, hop(y)), 0.0)
            al = (q.conj() * r).flatten(1).sum(1) / (q.conj() * q).flatten(1).sum(1)
            al = al[:, None, None, None, None, None, None]
            z, r = z + al * r, r - al * q
        mid = (slice(None),) + (slice(1, e - 1),) * 4
        out = torch.zeros_like(site)
        out[idx[mid].reshape(-1)] = z[mid].reshape(-1, 4, 3)
        return out.reshape(v.shape)


def exact(c, seed):
    U, vec = _fields(c, seed)
    dims, kind, kappa = _dims_of(c), c["kind"], c["kappa"]

    def grid(a):
        return a.reshape(*a.shape[:-3], *dims[::-1], 4, 3)

    if kind in ("grad", "train"):
        if kind == "train":
            w = _Wilson(dims, U, kappa)
            x = w.solve(grid(vec[0]))
            g5 = torch.tensor([1.0, 1, -1, -1], dtype=torch.complex128, device="cuda")[:, None]
            y = g5 * w.solve(g5 * grid(vec[1]))
        else:
            x, y = grid(vec[0]), grid(vec[1])
        U = U.detach().requires_grad_(True)
        kap = torch.tensor(kappa, dtype=torch.float64, device="cuda", requires_grad=True)
        loss = -(y.conj() * _Wilson(dims, U, kap).D(x)).real.sum()
        gU, gk = torch.autograd.grad(loss, (U, kap))
        if kind == "grad":
            return {"gU": gU, "gkappa": float(gk)}
        return {"x": x.reshape(vec[0].shape), "gU": gU, "gkappa": gk, "gb": y.reshape(vec[1].shape)}
    w = _Wilson(dims, U, kappa)
    v = vec[0]
    one = v.dim() == 3
    out = torch.empty_like(v)
    if kind == "solve":
        return w.solve(grid(v)).reshape(v.shape)
    ti = w.inv() if kind == "op" and c["op"] in ("clover_inv", "schur") else None
    even = w.parity() == 0
    for src, dst in [(v, out)] if one else zip(v, out):
        p = grid(src)
        if kind == "gauge" or kind == "apply":
            r = w.Ddag(p) if c.get("dagger") else w.D(p)
        elif c["op"] == "hop":
            r = w.hop(p)
        elif c["op"] == "clover_inv":
            r = w.chiral(ti, p)
        elif c["op"] == "schur":
            e = torch.where(even, p, 0.0)
            y = torch.where(even, 0.0, w.chiral(ti, w.hop(e)))
            r = e - kappa ** 2 * torch.where(even, w.chiral(ti, w.hop(y)), 0.0)
        else:
            r = torch.where(even, w.ras(p), 0.0)
        dst.copy_(r.reshape(src.shape))
    return out
