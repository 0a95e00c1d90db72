"""Timing cases: what a program that uses this library has it do, through the
public entry points (``Lattice``, ``CloverForce``), from single small operator
calls to a whole molecular-dynamics step on the largest lattice.

``listed`` names the cases, ``draw`` gives another of the same ranges,
``prepare`` makes what the program has in hand before the call (fields on the
GPU, the lattice context), ``run`` is one call and its outputs, ``work`` the
bytes and flops the call cannot do without, and ``exact`` the call's outputs
from plain complex128 tensor operations written out below.
"""
import math

import torch

from paper_0910_0262_amd import CloverForce, Lattice

C128, F64 = torch.complex128, torch.float64
DEV = "cuda"

# Link width -> (kappa, CG iterations to 1e-10, roughly): the roughness and
# masses of the synthetic workloads.  The iteration counts enter ``work`` only.
ROUGHNESS = {0.2: (0.1255, 140), 0.3: (0.125, 60), 0.5: (0.124, 45)}
KINDS = ("apply", "solve", "multi", "force", "config", "gauge", "det", "quenched", "trajectory")


def case(kind, dims, width, **more):
    lx, ly, lz, lt = dims
    return dict({"kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, "width": width, "kappa": ROUGHNESS[width][0], "csw": 1.0}, **more)


def listed():
    return [
        # one operator application on the smallest lattice: a call's own latency
        dict(case("apply", (4, 4, 4, 4), 0.3, op="M", prec="fp64"), name="apply M 4^4"),
        # the operator alone on the largest lattice, as measurement programs call it
        dict(case("apply", (32, 32, 32, 64), 0.2, op="MdagM", prec="fp64"), name="apply MdagM 32^3x64"),
        # a propagator source on the paper's smaller lattice, double precision throughout
        dict(case("solve", (8, 8, 16, 16), 0.5, prec="fp64", tol=1e-10), name="solve fp64 8x8x16x16"),
        # a propagator source on the paper's larger lattice, mixed precision
        dict(case("solve", (16, 16, 16, 16), 0.3, prec="mixed", tol=1e-10), name="solve mixed 16^4"),
        # three colours of one spin solved together (a count that is no power of two)
        dict(case("multi", (16, 16, 16, 16), 0.3, prec="fp64", tol=1e-10, n=3), name="multi fp64 3x16^4"),
        # eight sources on a lattice far larger than the caches: production propagators
        dict(case("multi", (32, 32, 32, 64), 0.2, prec="mixed", tol=1e-10, n=8), name="multi mixed 8x32^3x64"),
        # pseudofermion action and its gradient through autograd, forward and backward
        dict(case("force", (16, 16, 16, 16), 0.3, prec="fp64", tol=1e-12), name="force 16^4"),
        # a new configuration: load, build the clover term, apply the operator once
        dict(case("config", (32, 32, 32, 64), 0.2), name="config 32^3x64"),
        # the Wilson gauge action with its gradient and su(3) force
        dict(case("gauge", (32, 32, 32, 64), 0.2, beta=5.6), name="gauge force 32^3x64"),
        # the clover determinant's action, gradient and force
        dict(case("det", (24, 24, 24, 48), 0.2), name="det force 24^3x48"),
        # pure-gauge trajectory (thermalising a start configuration): many short launches
        dict(case("quenched", (16, 16, 16, 16), 0.3, beta=5.6, dt=0.02, steps=10), name="quenched 16^4"),
        # one step of the two-flavour R-algorithm trajectory on the largest lattice
        dict(case("trajectory", (32, 32, 32, 64), 0.2, beta=5.6, dt=0.02, steps=1, prec="mixed", tol=1e-10), name="trajectory 32^3x64"),
    ]


def _dims_of(rng, v_min, v_max):
    """Even extents with a volume spread over the logarithm of the range; odd aspect ratios included."""
    target = math.exp(rng.uniform(math.log(v_min), math.log(v_max)))
    while True:
        side = target ** 0.25
        d = [max(2, 2 * round(side * math.exp(rng.uniform(-0.4, 0.4)) / 2)) for _ in range(3)]
        d.append(max(2, 2 * round(target / (d[0] * d[1] * d[2]) / 2)))
        v = d[0] * d[1] * d[2] * d[3]
        if v_min <= v <= v_max and d[3] <= 96:
            return tuple(d)


def draw(rng):
    # the largest call of a kind: eight mixed sources, or about the same time
    # in double precision, on 32^3x64
    v32 = 32 ** 3 * 64
    kind = rng.choice(KINDS)
    width = rng.choice(sorted(ROUGHNESS))
    prec = rng.choice(("fp64", "mixed"))
    if kind == "apply":
        op = rng.choice(("M", "Mdag", "Mhat", "Mhatdag", "MdagM"))
        return case(kind, _dims_of(rng, 64, v32), width, op=op, prec="fp64" if op in ("M", "Mdag") else prec)
    if kind == "solve":
        return case(kind, _dims_of(rng, 256, v32 * 9 // 10), width, prec=prec, tol=1e-10)
    if kind == "multi":
        n = rng.randint(2, 16)
        slots = 1 << (n - 1).bit_length()
        return case(kind, _dims_of(rng, 256, min(v32, 8 * v32 // slots) // (5 if prec == "fp64" else 1)), width, prec=prec, tol=1e-10, n=n)
    if kind == "force":
        return case(kind, _dims_of(rng, 256, v32 // 2), width, prec=prec, tol=1e-12)
    if kind == "config":
        return case(kind, _dims_of(rng, 256, v32), width)
    if kind == "gauge":
        return case(kind, _dims_of(rng, 256, v32), width, beta=rng.choice((5.4, 5.6, 6.0)))
    if kind == "det":
        return case(kind, _dims_of(rng, 256, v32), width)
    if kind == "quenched":
        return case(kind, _dims_of(rng, 256, v32 // 2), width, beta=rng.choice((5.4, 5.6, 6.0)), dt=0.02, steps=rng.randint(1, 10))
    return case(kind, _dims_of(rng, 256, v32 * 9 // 10), width, beta=5.6, dt=0.02, steps=1, prec=prec, tol=1e-10)


# ------------------------------------------------------------------ inputs
def _dims(c):
    return (c["lx"], c["ly"], c["lz"], c["lt"])


def _volume(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _mm(a, b):
    """3x3 products of two fields of matrices."""
    return sum(a[..., :, k, None] * b[..., k, None, :] for k in range(3))


def _dag(a):
    return a.conj().transpose(-1, -2)


def _expi(h):
    """exp(i h) of Hermitian 3x3 matrices: Taylor series of h / 16, squared four times."""
    x = 1j * h / 16
    eye = torch.eye(3, dtype=C128, device=h.device)
    out = eye + x / 12
    for k in range(11, 0, -1):
        out = eye + _mm(x, out) / k
    for _ in range(4):
        out = _mm(out, out)
    return out


def _unitarize(u):
    a = u[..., 0, :]
    a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
    b = u[..., 1, :]
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack([a, b, torch.linalg.cross(a, b, dim=-1).conj()], dim=-2)


def _inputs(c, seed):
    """The fields the call starts from: SU(3) links of the case's roughness, Gaussian vectors and momenta."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    lx, ly, lz, lt = _dims(c)
    v = _volume(c)

    def normal(shape):
        return torch.view_as_complex(torch.randn(shape + (2,), dtype=F64, device=DEV, generator=gen))

    a = c["width"] * normal((lt, lz, ly, lx, 4, 3, 3))
    h = (a + _dag(a)) / 2
    h = h - torch.diagonal(h, dim1=-2, dim2=-1).mean(-1)[..., None, None] * torch.eye(3, dtype=C128, device=DEV)
    f = {"U": _unitarize(_expi(h)).contiguous()}
    del a, h
    kind = c["kind"]
    if kind == "apply":
        f["psi"] = normal((lt, lz, ly, lx, 4, 3) if c["op"] in ("M", "Mdag") else (v // 2, 4, 3))
    elif kind == "config":
        f["psi"] = normal((v // 2, 4, 3))
    elif kind == "solve":
        f["b"] = normal((lt, lz, ly, lx, 4, 3))
    elif kind == "multi":
        f["b"] = normal((c["n"], lt, lz, ly, lx, 4, 3))
    elif kind == "force":
        f["phi"] = normal((v // 2, 4, 3))
    elif kind in ("quenched", "trajectory"):
        f["P"] = torch.randn((lt, lz, ly, lx, 4, 8), dtype=F64, device=DEV, generator=gen)
        if kind == "trajectory":
            f["xi"] = normal((c["steps"], v // 2, 4, 3)) / math.sqrt(2)
    return f


def prepare(c, seed):
    s = _inputs(c, seed)
    s["case"] = c
    s["lat"] = Lattice(_dims(c), c["kappa"], c["csw"])
    if c["kind"] in ("apply", "solve", "multi", "det"):
        s["lat"].load_gauge(s["U"])
    elif c["kind"] == "gauge":
        s["lat"].load_gauge(s["U"], build_clover=False)
    return s


# ------------------------------------------------------------------ the calls
def run(s):
    c, lat = s["case"], s["lat"]
    kind = c["kind"]
    if kind == "apply":
        return lat.apply(c["op"], s["psi"], prec=c["prec"])
    if kind == "solve":
        return lat.solve(s["b"], prec=c["prec"], tol=c["tol"])[0]
    if kind == "multi":
        return lat.solve_multi(s["b"], prec=c["prec"], tol=c["tol"])[0]
    if kind == "config":
        lat.load_gauge(s["U"])
        return lat.apply("Mhat", s["psi"])
    if kind == "force":
        u, phi = s["U"].detach().requires_grad_(True), s["phi"].detach().requires_grad_(True)
        action = CloverForce.apply(u, phi, lat, c["prec"], c["tol"])
        action.backward()
        return {"S": action.detach(), "grad_U": u.grad, "grad_phi": phi.grad}
    if kind == "gauge":
        action, g, f = lat.gauge_action_force(c["beta"])
        return {"S": action, "G": g, "F": f}
    if kind == "det":
        action, g, f = lat.clover_det_action_force()
        return {"S": action, "G": g, "F": f}
    # the trajectory moves U and P in place; the program keeps its start
    # configuration (to repeat or to reject the trajectory)
    u, p = s["U"].clone(), s["P"].clone()
    if kind == "quenched":
        actions, _ = lat.md_trajectory(u, p, None, c["dt"], c["steps"], beta=c["beta"], n_f=0.0, reunitarize=True)
    else:
        actions, _ = lat.md_trajectory(u, p, s["xi"], c["dt"], c["steps"], beta=c["beta"], n_f=2.0, clover_det=True,
                                       reunitarize=True, prec=c["prec"], tol=c["tol"])
    return {"U": u, "P": p, "actions": [list(a) for a in actions]}


# ------------------------------------------------------------------ the least work
def _mdagm(c, n, prec):
    """Bytes and flops of one Mhat^dag Mhat on n vectors: four hops, each reading the links (two rows) and a
    clover block once, its input vectors once and writing its output (binary16 storage where mixed)."""
    vh = _volume(c) // 2
    sp, links, inv, ee = (192, 8 * 96, 576, 416) if prec == "fp64" else (52, 8 * 24, 152, 112)
    return {"bytes": 2 * vh * (5 * n * sp + 2 * links + inv + ee), "flops": 2 * 1824 * 2 * vh * n}


def _solve_work(c, n, prec, tol):
    m = _mdagm(c, n, prec)
    its = ROUGHNESS[c["width"]][1] * math.log(tol) / math.log(1e-10)
    sp = 192 if prec == "fp64" else 52
    vectors = 2 * 192 * _volume(c) * n
    return {"bytes": its * (m["bytes"] + 5 * sp * _volume(c) // 2 * n) + vectors, "flops": its * m["flops"]}


def work(c):
    v = _volume(c)
    kind = c["kind"]
    u, g, f, clover = 576 * v, 576 * v, 256 * v, 576 * v
    mm = 198 * v  # one 3x3 complex product per site
    if kind == "apply":
        m = _mdagm(c, 1, c["prec"])
        share = 0.5 if c["op"] != "MdagM" else 1.0
        return {"bytes": share * m["bytes"], "flops": share * m["flops"]}
    if kind == "solve":
        return _solve_work(c, 1, c["prec"], c["tol"])
    if kind == "multi":
        return _solve_work(c, c["n"], c["prec"], c["tol"])
    if kind == "config":
        m = _mdagm(c, 1, "fp64")
        return {"bytes": u + 1.5 * clover + 0.5 * m["bytes"], "flops": 72 * mm + 0.5 * m["flops"]}
    if kind == "gauge":
        return {"bytes": u + g + f, "flops": 4 * 13 * mm + 12 * mm}
    if kind == "det":
        return {"bytes": u + clover / 2 + g + f, "flops": 4 * 42 * mm}
    if kind == "force":
        w = _solve_work(c, 1, c["prec"], c["tol"])
        return {"bytes": w["bytes"] + u + 1.5 * clover + g, "flops": w["flops"] + 4 * 42 * mm + 72 * mm}
    step = {"bytes": 4 * u + 3 * f, "flops": 4 * 13 * mm + 12 * mm + 8 * 6 * mm}
    if kind == "trajectory":
        w = _solve_work(c, 1, c["prec"], c["tol"])
        step = {"bytes": step["bytes"] + w["bytes"] + 3 * clover, "flops": step["flops"] + w["flops"] + 4 * 42 * mm + 144 * mm}
    return {k: c["steps"] * step[k] for k in step}


# ------------------------------------------------------------------ the same outputs in plain complex128
# gamma_mu psi in the chiral basis: spin s of the product is PHASE[mu][s] psi[PERM[mu][s]]
PERM = ((3, 2, 1, 0), (3, 2, 1, 0), (2, 3, 0, 1), (2, 3, 0, 1))
PHASE = ((-1j, -1j, 1j, 1j), (-1, 1, 1, -1), (-1j, 1j, 1j, -1j), (1, 1, 1, 1))


def _gamma(mu, psi):
    return psi[..., list(PERM[mu]), :] * torch.tensor(PHASE[mu], dtype=C128, device=psi.device)[:, None]


def _gamma_matrix(mu):
    g = torch.zeros(4, 4, dtype=C128, device=DEV)
    for s in range(4):
        g[s, PERM[mu][s]] = PHASE[mu][s]
    return g


def _at(f, mu, n=1):
    """f(x + n mu)."""
    return torch.roll(f, -n, 3 - mu)


def _site_mv(u, psi):
    """u psi on colour, for every spin."""
    return sum(u[..., None, :, k] * psi[..., :, k, None] for k in range(3))


def _hop(u, psi, sign=1.0):
    """H psi on the whole lattice, antiperiodic in time; sign = -1 for H^dag."""
    out = torch.zeros_like(psi)
    for mu in range(4):
        um = u[..., mu, :, :]
        fwd, bwd = _at(psi, mu), _at(_site_mv(_dag(um), psi), mu, -1)
        if mu == 3:
            fwd = torch.cat([fwd[:-1], -fwd[-1:]])
            bwd = torch.cat([-bwd[:1], bwd[1:]])
        fwd = _site_mv(um, fwd)
        out = out + fwd + bwd - sign * _gamma(mu, fwd - bwd)
    return out


def _clover_blocks(u, kc):
    """A = 1 - kappa c_sw sum sigma F as its two 6x6 blocks, (T, Z, Y, X, 2, 6, 6)."""
    eye3 = torch.eye(3, dtype=C128, device=u.device)
    blocks = torch.eye(6, dtype=C128, device=u.device).expand(u.shape[:4] + (2, 6, 6))
    for mu in range(4):
        for nu in range(mu + 1, 4):
            um, un = u[..., mu, :, :], u[..., nu, :, :]
            # the plaquette from each of its corners is the same loop carried along its links
            a, b = _mm(um, _at(un, mu)), _mm(un, _at(um, nu))
            q = _mm(a, _dag(b))                                          # from x
            p = _mm(_dag(un), _mm(a, _dag(_at(um, nu))))                 # from x + nu
            q = q + _at(p, nu, -1)
            p = _mm(_mm(_at(un, mu), _dag(b)), um)                       # from x + mu
            q = q + _at(p, mu, -1)
            p = _mm(_dag(b), a)                                          # from x + mu + nu
            q = q + _at(_at(p, mu, -1), nu, -1)
            f = (q - _dag(q)) / 8j
            f = f - torch.diagonal(f, dim1=-2, dim2=-1).mean(-1)[..., None, None] * eye3
            g1, g2 = _gamma_matrix(mu), _gamma_matrix(nu)
            sigma = 0.5j * (g1 @ g2 - g2 @ g1)
            for k in range(2):
                s = sigma[2 * k:2 * k + 2, 2 * k:2 * k + 2]
                kron = (s[:, None, :, None] * f[..., None, :, None, :]).reshape(u.shape[:4] + (6, 6))
                part = torch.zeros(2, 1, 1, dtype=C128, device=u.device)
                part[k] = kc
                blocks = blocks - part * kron[..., None, :, :]
    return blocks


def _inverse(a):
    """Inverse of positive definite matrices by elimination."""
    n = a.shape[-1]
    m = torch.cat([a, torch.eye(n, dtype=a.dtype, device=a.device).expand_as(a)], -1)
    for j in range(n):
        row = m[..., j, :] / m[..., j, j, None]
        m = m - m[..., :, j, None] * row[..., None, :]
        m[..., j, :] = row
    return m[..., n:].contiguous()


def _logdet(a):
    total = 0.0
    while a.shape[-1] > 0:
        p = a[..., 0, 0].real
        total = total + torch.log(p)
        a = a[..., 1:, 1:] - a[..., 1:, :1] * a[..., :1, 1:] / p[..., None, None]
    return total


class _Operators:
    """The even-odd operators on whole-lattice vectors that vanish off their parity."""

    def __init__(self, u, kappa, csw):
        lt, lz, ly, lx = u.shape[:4]
        self.u, self.kappa = u, kappa
        axes = [torch.arange(n, device=u.device).view([n if k == j else 1 for k in range(4)]) for j, n in enumerate((lt, lz, ly, lx))]
        par = (axes[0] + axes[1] + axes[2] + axes[3]) % 2
        self.odd = par.bool()
        self.even_sites = torch.nonzero(par.reshape(-1) == 0).reshape(-1)
        self.A = _clover_blocks(u, kappa * csw)
        self.Ainv = _inverse(self.A)

    def parity(self, psi, odd):
        return psi * (self.odd if odd else ~self.odd)[..., None, None]

    def block(self, a, psi):
        v = psi.reshape(psi.shape[:-2] + (2, 6))
        return sum(a[..., :, k] * v[..., k, None] for k in range(6)).reshape(psi.shape)

    def spread(self, e):
        full = torch.zeros(self.odd.shape + (4, 3), dtype=C128, device=e.device)
        full.view(-1, 4, 3)[self.even_sites] = e
        return full

    def gather(self, full):
        return full.reshape(-1, 4, 3)[self.even_sites]

    def M(self, psi, sign=1.0):
        return self.block(self.A, psi) - self.kappa * _hop(self.u, psi, sign)

    def mhat(self, e, sign=1.0):
        t = self.parity(self.block(self.Ainv, _hop(self.u, e, sign)), True)
        return self.parity(self.block(self.A, e) - self.kappa ** 2 * _hop(self.u, t, sign), False)

    def normal_solve(self, rhs, tol=1e-13):
        x = torch.zeros_like(rhs)
        r, p = rhs.clone(), rhs.clone()
        rr = stop = float((r.conj() * r).sum().real)
        for k in range(2000):
            if rr <= tol * tol * stop:
                break
            q = self.mhat(p)
            a = rr / float((q.conj() * q).sum().real)
            x = x + a * p
            # the recurrence's residual, recomputed now and then
            r = r - a * self.mhat(q, -1.0) if k % 50 != 49 else rhs - self.mhat(self.mhat(x), -1.0)
            new = float((r.conj() * r).sum().real)
            p = r + (new / rr) * p
            rr = new
        return x

    def solve(self, b):
        bo = self.parity(b, True)
        bhat = self.parity(b + self.kappa * _hop(self.u, self.block(self.Ainv, bo)), False)
        e = self.normal_solve(self.mhat(bhat, -1.0))
        return e + self.parity(self.block(self.Ainv, bo + self.kappa * _hop(self.u, e)), True)

    def action_gradient(self, phi, csw):
        """phi^dag (Mhat^dag Mhat)^-1 phi on even sites, its gradient in the links, and the solution."""
        x = self.normal_solve(phi)
        y = self.mhat(x)
        z = self.parity(self.block(self.Ainv, _hop(self.u, x)), True)
        w = self.parity(self.block(self.Ainv, _hop(self.u, y, -1.0)), True)
        # dS = -2 Re[y^dag dMhat x], with A_oo^-1 differentiated into the odd parts w and z
        u = self.u.detach().clone().requires_grad_(True)
        a = _clover_blocks(u, self.kappa * csw)
        k2 = self.kappa ** 2
        dot = (y.conj() * (self.block(a, x) - k2 * _hop(u, z))).sum() - k2 * (w.conj() * _hop(u, x)).sum() \
            + k2 * (w.conj() * self.block(a, z)).sum()
        (grad,) = torch.autograd.grad(-2.0 * dot.real, u)
        return float((phi.conj() * x).sum().real), grad, x


def _gradient(action, u):
    u = u.detach().clone().requires_grad_(True)
    s = action(u)
    (grad,) = torch.autograd.grad(s, u)
    return float(s.detach()), grad


def _gauge_action(u, beta):
    s = 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a = _mm(u[..., mu, :, :], _at(u[..., nu, :, :], mu))
            b = _mm(u[..., nu, :, :], _at(u[..., mu, :, :], nu))
            s = s + (1.0 - (a * b.conj()).real.sum((-1, -2)) / 3.0).sum()
    return beta * s


def _det_action(u, kc, odd):
    return -2.0 * (_logdet(_clover_blocks(u, kc)).sum(-1) * odd).sum()


def _generators():
    lam = torch.zeros(8, 3, 3, dtype=C128, device=DEV)
    lam[0, 0, 1] = lam[0, 1, 0] = 1
    lam[1, 0, 1], lam[1, 1, 0] = -1j, 1j
    lam[2, 0, 0], lam[2, 1, 1] = 1, -1
    lam[3, 0, 2] = lam[3, 2, 0] = 1
    lam[4, 0, 2], lam[4, 2, 0] = -1j, 1j
    lam[5, 1, 2] = lam[5, 2, 1] = 1
    lam[6, 1, 2], lam[6, 2, 1] = -1j, 1j
    lam[7, 0, 0] = lam[7, 1, 1] = 1 / math.sqrt(3)
    lam[7, 2, 2] = -2 / math.sqrt(3)
    return lam / 2


def _su3_force(u, g):
    """F^a = Re(i tr[T^a U G^dag])."""
    w = _mm(u, _dag(g))
    return torch.stack([-(t.transpose(0, 1) * w).sum((-1, -2)).imag for t in _generators()], -1)


def _move(u, p, h):
    return _mm(_expi(sum(h * p[..., a, None, None] * t for a, t in enumerate(_generators()))), u)


def exact(c, seed):
    kind, v = c["kind"], _volume(c)
    vectors = v * c.get("n", 1)
    # solves of the largest lattices take longer here than is worth it
    if kind in ("solve", "multi", "force", "trajectory") and vectors * ROUGHNESS[c["width"]][1] > 6e7:
        return None
    f = _inputs(c, seed)
    u, kappa, csw = f["U"], c["kappa"], c["csw"]
    if kind == "gauge":
        s, g = _gradient(lambda w: _gauge_action(w, c["beta"]), u)
        return {"S": s, "G": g, "F": _su3_force(u, g)}
    if kind == "quenched":
        p, actions = f["P"], []
        for _ in range(c["steps"]):
            u = _move(u, p, 0.5 * c["dt"])
            s, g = _gradient(lambda w: _gauge_action(w, c["beta"]), u)
            actions.append([0.0, s, 0.0])
            p = p - c["dt"] * _su3_force(u, g)
            u = _unitarize(_move(u, p, 0.5 * c["dt"]))
        return {"U": u, "P": p, "actions": actions}
    ops = _Operators(u, kappa, csw)
    if kind == "apply":
        if c["prec"] != "fp64":
            return None  # binary16 storage: the outputs carry its rounding
        sign = -1.0 if c["op"] in ("Mdag", "Mhatdag") else 1.0
        if c["op"] in ("M", "Mdag"):
            return ops.M(f["psi"], sign)
        e = ops.mhat(ops.spread(f["psi"]), sign)
        return ops.gather(ops.mhat(e, -1.0) if c["op"] == "MdagM" else e)
    if kind == "config":
        return ops.gather(ops.mhat(ops.spread(f["psi"])))
    if kind == "solve":
        return ops.solve(f["b"])
    if kind == "multi":
        return torch.stack([ops.solve(b) for b in f["b"]])
    if kind == "force":
        s, g, x = ops.action_gradient(ops.spread(f["phi"]), csw)
        return {"S": s, "grad_U": g, "grad_phi": 2.0 * ops.gather(x)}
    if kind == "det":
        s, g = _gradient(lambda w: _det_action(w, kappa * csw, ops.odd), u)
        return {"S": s, "G": g, "F": _su3_force(u, g)}
    p, actions = f["P"], []
    for xi in f["xi"]:  # two flavours: the noise is drawn where the step starts
        phi = _Operators(u, kappa, csw).mhat(ops.spread(xi), -1.0)
        u = _move(u, p, 0.5 * c["dt"])
        s_f, g, _ = _Operators(u, kappa, csw).action_gradient(phi, csw)
        s_g, g_g = _gradient(lambda w: _gauge_action(w, c["beta"]), u)
        s_d, g_d = _gradient(lambda w: _det_action(w, kappa * csw, ops.odd), u)
        actions.append([s_f, s_g, s_d])
        p = p - c["dt"] * _su3_force(u, g + g_g + g_d)
        u = _unitarize(_move(u, p, 0.5 * c["dt"]))
    return {"U": u, "P": p, "actions": actions}
