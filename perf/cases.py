"""The work that users of this package have it do, as measurable cases.

Each case is one call through the package's public entry points (`Hubbard`,
`Batch`) on a seeded problem of the kind its workloads and tests use:
Hubbard clusters at half filling from the checkerboard state, circuit
parameters ~ U(-pi/8, pi/8), hopping disorder 1 + 0.1 N(0, 1), on-site
energies ~ U(-0.5, 0.5) and a nearest-neighbour V.  `exact` computes the same
results with plain torch operations in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2408_00836_amd import workloads as W
from paper_2408_00836_amd.model import Batch, Hubbard

U_DEFAULT = 4.0
V_DEFAULT = 0.5


def _case(op, nx, ny, layers, *, px=False, py=False, general=False, U=U_DEFAULT, count=0,
          name=None):
    c = dict(op=op, nx=nx, ny=ny, px=px, py=py, general=general, U=float(U), layers=layers,
             count=count)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a 2x2 cluster inside an optimiser's loop, all latency
        _case("energy_grad", 2, 2, 2, name="grad_2x2_8q"),
        # an ordinary chain (the paper's 1D study), 16 qubits
        _case("energy_grad", 1, 8, 8, name="grad_1x8_16q"),
        # the inhomogeneous ladder with disorder, on-site energies and V, 24 qubits
        _case("energy_grad", 2, 6, 12, general=True, name="grad_2x6_general_24q"),
        # a large full vector: 4 GiB for psi, the same for lambda
        _case("energy_grad", 2, 7, 4, name="grad_2x7_28q"),
        # state preparation (forward only) that hands the whole vector to the user
        _case("ansatz", 2, 6, 6, name="state_2x6_24q"),
        # H on a user's full vector, as a Krylov or time-evolution loop calls it
        _case("apply_h", 2, 7, 0, name="h_2x7_28q"),
        # the number-preserving ansatz: one parameter pair per coupled qubit pair
        _case("np_grad", 3, 3, 3, U=2.0, name="np_3x3_18q"),
        # the uneven batch: 256 instances, 8-20 qubits, every one with disorder
        _case("batch", 0, 0, 0, count=256, name="batch_256"),
        # the sector form of the 4x4 torus, the largest lattice
        _case("sector_grad", 4, 4, 8, px=True, py=True, U=8.0, name="sector_4x4_32q"),
        # the sector form of the inhomogeneous ladder
        _case("sector_grad", 2, 6, 12, general=True, name="sector_2x6_general_24q"),
        # the sector form of a chain: short rows, many calls of a VQE run
        _case("sector_grad", 1, 10, 8, name="sector_1x10_20q"),
        # H on a sector vector of the torus, the step of the Lanczos reference
        _case("sector_h", 4, 4, 0, px=True, py=True, U=8.0, name="sector_h_4x4_32q"),
    ]


# Lattices by operation: (nx, ny, periodic_x, periodic_y).
_SMALL = [(1, 2, 0, 0), (1, 3, 0, 0), (1, 4, 0, 1), (2, 2, 0, 0), (1, 5, 0, 0), (2, 3, 0, 0),
          (1, 6, 0, 1)]
_MIDDLE = [(1, 7, 0, 0), (2, 4, 0, 0), (1, 8, 0, 1), (3, 3, 0, 0), (1, 9, 0, 0), (2, 5, 0, 0),
           (1, 10, 0, 0)]
_LARGE = [(1, 11, 0, 0), (3, 4, 0, 1), (2, 6, 0, 0), (1, 12, 0, 0), (1, 13, 0, 0)]
_SECTOR = [(2, 4, 0, 0), (1, 9, 0, 0), (3, 3, 0, 0), (2, 5, 0, 0), (1, 11, 0, 0), (3, 4, 0, 1),
           (2, 6, 0, 0), (1, 13, 0, 0), (2, 7, 0, 0), (3, 5, 0, 0), (1, 14, 0, 1)]
_SECTOR_TOP = [(4, 4, 0, 0), (4, 4, 1, 1), (2, 8, 0, 0), (1, 16, 0, 0), (1, 15, 0, 0)]


def draw(rng):
    op = rng.choice(["energy_grad", "energy_grad", "energy_grad", "ansatz", "apply_h", "np_grad",
                     "batch", "sector_grad", "sector_grad", "sector_grad", "sector_h"])
    U = round(rng.uniform(1.0, 8.0), 3)
    general = rng.random() < 0.4
    if op == "batch":
        return _case(op, 0, 0, 0, count=int(round(math.exp(rng.uniform(math.log(3), math.log(200))))))
    if op == "np_grad":
        nx, ny, px, py = rng.choice(_SMALL + _MIDDLE)
        return _case(op, nx, ny, rng.randint(1, 3), px=bool(px), py=bool(py), general=general, U=U)
    if op == "sector_grad":
        top = rng.random() < 0.25
        nx, ny, px, py = rng.choice(_SECTOR_TOP if top else _SECTOR)
        return _case(op, nx, ny, rng.randint(1, 5 if top else 10), px=bool(px), py=bool(py),
                     general=general and not top, U=U)
    if op == "sector_h":
        nx, ny, px, py = rng.choice(_SECTOR + _SECTOR_TOP)
        return _case(op, nx, ny, 0, px=bool(px), py=bool(py), general=general, U=U)
    nx, ny, px, py = rng.choice(rng.choice([_SMALL, _MIDDLE, _LARGE]))
    layers = 0 if op == "apply_h" else rng.randint(1, 10)
    return _case(op, nx, ny, layers, px=bool(px), py=bool(py), general=general, U=U)


# ------------------------------------------------------------------ inputs --

def _n_bonds(c):
    return W.n_bonds(c["nx"], c["ny"], c["px"], c["py"])


def _coefficients(c, rng):
    """t per bond, V per bond, eps per site (None: uniform t = 1, no V, no eps)."""
    if not c["general"]:
        return None, None, None
    nb = _n_bonds(c)
    return (1.0 + 0.1 * rng.standard_normal(nb), np.full(nb, V_DEFAULT),
            rng.uniform(-0.5, 0.5, c["nx"] * c["ny"]))


def _angles(rng, n):
    return rng.uniform(-np.pi / 8, np.pi / 8, n)


def _problem(c, seed):
    """(host inputs of a single-instance case): coefficients and a generator
    that goes on with the angles or the vector's seed."""
    rng = np.random.default_rng(seed)
    t, V, eps = _coefficients(c, rng)
    return rng, t, V, eps


def _vector(c, seed, n):
    """A user's unit vector of n amplitudes."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    v = torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g)
    v /= torch.linalg.vector_norm(v)
    return torch.view_as_complex(v)


def _batch_workloads(c, seed):
    ws = W.batch(c["count"])
    rng = np.random.default_rng(seed)
    for w in ws:
        w.theta = _angles(rng, w.theta.size)
    return ws


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    s.op = c["op"]
    if s.op == "batch":
        ws = _batch_workloads(c, seed)
        s.models = [Hubbard(w.nx, w.ny, **w.kwargs()) for w in ws]
        s.batch = Batch(s.models, [w.layers for w in ws])
        s.theta = torch.tensor(np.concatenate([w.theta for w in ws]), device="cuda")
        return s
    rng, t, V, eps = _problem(c, seed)
    s.model = Hubbard(c["nx"], c["ny"], periodic_x=c["px"], periodic_y=c["py"], t=t, U=c["U"],
                      V=V, eps=eps, ansatz="np" if s.op == "np_grad" else "hva")
    if s.op == "apply_h":
        s.psi = _vector(c, seed, s.model.dim)
        s.out = torch.empty_like(s.psi)
    elif s.op == "sector_h":
        nu, nd = s.model.sector_dims()
        s.psi = _vector(c, seed, nu * nd)
        s.out = torch.empty_like(s.psi)
    else:
        s.theta = torch.tensor(_angles(rng, s.model.n_params(c["layers"])), device="cuda")
    return s


def run(state):
    s = state
    if s.op in ("energy_grad", "np_grad"):
        return s.model.energy_grad(s.theta)
    if s.op == "sector_grad":
        return s.model.sector_energy_grad(s.theta)
    if s.op == "ansatz":
        return s.model.ansatz(s.theta)
    if s.op == "apply_h":
        return s.model.apply_h(s.psi, s.out)
    if s.op == "sector_h":
        return s.model.sector_apply_h(s.psi, s.out)
    return s.batch.energy_grad(s.theta)


# ------------------------------------------------------------- work counts --

def _sector_sizes(nx, ny):
    up = sum(1 for x in range(nx) for y in range(ny) if (x + y) % 2 == 0)
    ns = nx * ny
    return math.comb(ns, up), math.comb(ns, ns - up)


def _circuit_flops(nx, ny, layers, nb, dim):
    """Forward, H and the adjoint sweep on `dim` amplitudes: a hopping gate
    rotates about half of them (12 operations a pair), the diagonal is one
    complex product each; the reverse does both for two vectors and reduces
    one bracket per term."""
    hop = dim / 4 * 12
    fwd = layers * (2 * nb * hop + 6 * dim)
    ham = 2 * nb * dim + 2 * dim
    rev = layers * (2 * nb * (2 * hop + dim / 4 * 8) + 16 * dim)
    return fwd, ham, rev


def work(case):
    c = case
    if c["op"] == "batch":
        b = f = 0.0
        for w in W.batch(c["count"]):
            nu, nd = _sector_sizes(w.nx, w.ny)
            nb = W.n_bonds(w.nx, w.ny, w.periodic_x, w.periodic_y)
            f += sum(_circuit_flops(w.nx, w.ny, w.layers, nb, float(nu * nd)))
            b += 8.0 * (2 * w.n_params + 1)
        return {"bytes": b, "flops": f}
    ns, nb, L = c["nx"] * c["ny"], _n_bonds(c), c["layers"]
    nu, nd = _sector_sizes(c["nx"], c["ny"])
    sector, full = float(nu * nd), float(4 ** ns)
    if c["op"] == "apply_h":
        return {"bytes": 32.0 * full, "flops": 2 * nb * full + 2 * full}
    if c["op"] == "sector_h":
        return {"bytes": 32.0 * sector, "flops": 2 * nb * sector + 2 * sector}
    if c["op"] == "np_grad":
        terms = ns + 2 * nb
        gate = full / 4 * 12 + full / 4 * 6
        return {"bytes": 8.0 * (2 * (2 * ns + 2 * terms * L) + 1),
                "flops": L * terms * (3 * gate + full / 4 * 12) + 2 * nb * full + 2 * full}
    fwd, ham, rev = _circuit_flops(c["nx"], c["ny"], L, nb, sector)
    params = 5 * L
    if c["op"] == "ansatz":
        return {"bytes": 16.0 * full + 8.0 * params, "flops": fwd}
    return {"bytes": 8.0 * (2 * params + 1), "flops": fwd + ham + rev}


# ------------------------------------------------- the same in plain torch --

def _lattice(nx, ny, px, py):
    """Bonds in canonical order with the rank of their hopping group in the
    order h1, v1, h2, v2: horizontal bonds split by the parity of their start
    column, vertical ones by that of their start row, the short direction of
    a ladder by the other coordinate."""
    bonds, key = [], []
    for x in range(nx):
        for y in range(ny):
            if y + 1 < ny or py:
                bonds.append((x * ny + y, x * ny + (y + 1) % ny))
                key.append(2 * ((x if ny == 2 and nx >= 3 else y) % 2))
    for x in range(nx):
        for y in range(ny):
            if x + 1 < nx or px:
                bonds.append((x * ny + y, (x + 1) % nx * ny + y))
                key.append(1 + 2 * ((y if nx == 2 and ny >= 3 else x) % 2))
    ids = sorted(set(key))
    return bonds, [1 + ids.index(k) for k in key], len(ids)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


class _Sector:
    """The circuit on the matrix of the start state's particle-number sector
    (rows: spin-down patterns, columns: spin-up patterns, both ascending)."""

    def __init__(self, nx, ny, px, py, U, t, V, eps):
        self.dev = dev = _device()
        ns = nx * ny
        self.bonds, self.slot, self.groups = _lattice(nx, ny, px, py)
        nb = len(self.bonds)
        t = np.ones(nb) if t is None else t
        V = np.zeros(nb) if V is None else V
        eps = np.zeros(ns) if eps is None else eps
        self.t = t
        even = [x * ny + y for x in range(nx) for y in range(ny) if (x + y) % 2 == 0]
        start = [sum(1 << s for s in range(ns) if (s in even) == up) for up in (True, False)]
        self.pats, bits, self.at, self.hop = [], [], [], []
        for spin in (0, 1):
            k = start[spin].bit_count()
            p = np.array([x for x in range(1 << ns) if x.bit_count() == k], dtype=np.int64)
            self.pats.append(p)
            bits.append(torch.tensor((p[:, None] >> np.arange(ns)) & 1, dtype=torch.float64,
                                     device=dev))
            self.at.append(int(np.searchsorted(p, start[spin])))
            per = []
            for i, j in self.bonds:
                lo, hi = min(i, j), max(i, j)
                act = ((p >> lo) ^ (p >> hi)) & 1
                to = np.where(act == 1, np.searchsorted(p, p ^ ((1 << lo) | (1 << hi))) % p.size,
                              np.arange(p.size))
                between = ((1 << hi) - 1) & ~((2 << lo) - 1)
                par = np.array([int(x).bit_count() & 1 for x in p & between])
                per.append((torch.tensor(to, device=dev),
                            torch.tensor(act * (1.0 - 2.0 * par), dtype=torch.float64,
                                         device=dev)))
            self.hop.append(per)
        w = np.zeros((ns, ns))
        for (i, j), v in zip(self.bonds, V):
            w[i, j] += v
            w[j, i] += v
        w = torch.tensor(w, device=dev)
        e = torch.tensor(np.asarray(eps, dtype=np.float64), device=dev)
        up, dn = bits
        one = [b @ e + 0.5 * ((b @ w) * b).sum(1) for b in bits]
        self.D = U * (dn @ up.T) + dn @ w @ up.T + one[1][:, None] + one[0][None, :]
        self.per = 1 + self.groups

    def start(self):
        psi = torch.zeros_like(self.D, dtype=torch.complex128)
        psi[self.at[1], self.at[0]] = 1.0
        return psi

    def swap(self, psi, spin, b):
        """(hopping operator without its -t) psi."""
        to, sgn = self.hop[spin][b]
        return psi[:, to] * sgn if spin == 0 else psi[to] * sgn[:, None]

    def rotate(self, psi, hpsi, spin, b, a):
        """exp(i a h) psi with hpsi = h psi, in place."""
        act = self.hop[spin][b][1].abs()
        cs = 1.0 + (math.cos(a) - 1.0) * act
        psi *= cs if spin == 0 else cs[:, None]
        return psi.add_(hpsi, alpha=complex(0.0, math.sin(a)))

    def gates(self, theta):
        for l in range(len(theta) // self.per):
            yield l * self.per, None, None
            for s in range(1, self.per):
                for b, sl in enumerate(self.slot):
                    if sl == s:
                        for spin in (0, 1):
                            yield l * self.per + s, spin, b

    def phase(self, psi, a):
        psi *= torch.polar(torch.ones_like(self.D), a * self.D)
        return psi

    def forward(self, theta):
        psi = self.start()
        for k, spin, b in self.gates(theta):
            if b is None:
                psi = self.phase(psi, -theta[k])
            else:
                psi = self.rotate(psi, self.swap(psi, spin, b), spin, b, theta[k] * self.t[b])
        return psi

    def ham(self, psi):
        out = self.D * psi
        for spin in (0, 1):
            for b in range(len(self.bonds)):
                out.add_(self.swap(psi, spin, b), alpha=-float(self.t[b]))
        return out

    def brackets(self, theta, psi, lam):
        """2 Im <lambda|G_k|psi> per parameter while both are un-applied."""
        g = [torch.zeros((), dtype=torch.float64, device=self.dev) for _ in theta]
        for k, spin, b in reversed(list(self.gates(theta))):
            if b is None:
                g[k] = g[k] + 2.0 * torch.vdot(lam.flatten(), (self.D * psi).flatten()).imag
                psi, lam = self.phase(psi, theta[k]), self.phase(lam, theta[k])
            else:
                a = -theta[k] * self.t[b]
                h = self.swap(psi, spin, b)
                g[k] = g[k] - 2.0 * self.t[b] * torch.vdot(lam.flatten(), h.flatten()).imag
                psi = self.rotate(psi, h, spin, b, a)
                lam = self.rotate(lam, self.swap(lam, spin, b), spin, b, a)
        return torch.stack(g)

    def grad(self, theta):
        psi = self.forward(theta)
        lam = self.ham(psi)
        E = torch.vdot(psi.flatten(), lam.flatten()).real.reshape(1)
        return E, self.brackets(theta, psi, lam)


class _Full:
    """Hopping terms and mask phases on all 2^n amplitudes."""

    def __init__(self, ns):
        self.n = 2 * ns
        self.idx = torch.arange(1 << self.n, device=_device())

    def bit(self, q):
        return (self.idx >> q) & 1

    def hop(self, p, q):
        """(partner index, sign or 0) of the hopping operator on qubits p, q."""
        lo, hi = min(p, q), max(p, q)
        par = torch.zeros_like(self.idx)
        for r in range(lo + 1, hi):
            par ^= self.bit(r)
        act = self.bit(lo) ^ self.bit(hi)
        return self.idx ^ ((1 << lo) | (1 << hi)), (act * (1 - 2 * par)).to(torch.float64)

    def diagonal(self, ns, bonds, U, V, eps):
        up, dn = ([self.bit(i + s).to(torch.float64) for i in range(ns)] for s in (0, ns))
        occ = [a + b for a, b in zip(up, dn)]
        d = torch.zeros(self.idx.numel(), dtype=torch.float64, device=self.idx.device)
        for i in range(ns):
            d += U * (up[i] * dn[i])
            if eps is not None:
                d += float(eps[i]) * occ[i]
        if V is not None:
            for (i, j), v in zip(bonds, V):
                d += float(v) * (occ[i] * occ[j])
        return d

    def ham(self, psi, ns, bonds, U, t, V, eps):
        out = self.diagonal(ns, bonds, U, V, eps) * psi
        for b, (i, j) in enumerate(bonds):
            for s in (0, ns):
                to, sgn = self.hop(i + s, j + s)
                out.add_(psi[to] * sgn, alpha=-1.0 if t is None else -float(t[b]))
                del to, sgn
        return out


def _np_grad(c, theta, t, V, eps):
    """Energy and adjoint gradient of the number-preserving circuit."""
    nx, ny = c["nx"], c["ny"]
    ns = nx * ny
    F = _Full(ns)
    bonds, slot, groups = _lattice(nx, ny, c["px"], c["py"])
    gates = [(q, None, (q,)) for q in range(2 * ns)]
    k = 2 * ns
    pairs = [(i, i + ns) for i in range(ns)]
    for s in range(1, groups + 1):
        for b, (i, j) in enumerate(bonds):
            if slot[b] == s:
                pairs += [(i, j), (i + ns, j + ns)]
    for _ in range(c["layers"]):
        for p, q in pairs:
            gates += [(k, (p, q), None), (k + 1, None, (p, q))]
            k += 2
    hops = {pq: F.hop(*pq) for pq in set(pairs)}

    def occupied(qs):
        m = torch.ones_like(F.idx)
        for q in qs:
            m = m & F.bit(q)
        return m.to(torch.float64)

    def apply(v, gate, a, h=None):
        """exp(i a h) v or exp(i a n..n) v."""
        _, pq, qs = gate
        if pq is None:
            return v * torch.polar(torch.ones_like(masks[qs]), a * masks[qs])
        to, sgn = hops[pq]
        h = v[to] * sgn if h is None else h
        return v * (1.0 + (math.cos(a) - 1.0) * sgn.abs()) + 1j * math.sin(a) * h

    masks = {g[2]: occupied(g[2]) for g in gates if g[2] is not None}
    even = [x * ny + y for x in range(nx) for y in range(ny) if (x + y) % 2 == 0]
    psi = torch.zeros(1 << F.n, dtype=torch.complex128, device=F.idx.device)
    psi[sum(1 << (s if s in even else s + ns) for s in range(ns))] = 1.0
    for g in gates:
        psi = apply(psi, g, theta[g[0]])
    lam = F.ham(psi, ns, bonds, c["U"], t, V, eps)
    E = torch.vdot(psi, lam).real.reshape(1)
    out = [None] * len(theta)
    for g in reversed(gates):
        _, pq, qs = g
        h = masks[qs] * psi if pq is None else psi[hops[pq][0]] * hops[pq][1]
        out[g[0]] = -2.0 * torch.vdot(lam, h).imag   # gate exp(+i th G): G enters with -1
        psi, lam = apply(psi, g, -theta[g[0]], h if pq else None), apply(lam, g, -theta[g[0]])
    return E, torch.stack(out)


def exact(case, seed):
    c = case
    if c["op"] == "batch":
        Es, gs = [], []
        for w in _batch_workloads(c, seed):
            S = _Sector(w.nx, w.ny, w.periodic_x, w.periodic_y, w.U, w.t, w.V, w.eps)
            E, g = S.grad(w.theta)
            Es.append(E)
            gs.append(g)
        return torch.cat(Es), torch.cat(gs)
    rng, t, V, eps = _problem(c, seed)
    nx, ny, ns, L = c["nx"], c["ny"], c["nx"] * c["ny"], c["layers"]
    if c["op"] == "apply_h":
        F = _Full(ns)
        return F.ham(_vector(c, seed, 1 << F.n), ns, _lattice(nx, ny, c["px"], c["py"])[0], c["U"],
                     t, V, eps)
    if c["op"] == "np_grad":
        terms = ns + 2 * _n_bonds(c)
        return _np_grad(c, _angles(rng, 2 * ns + 2 * terms * L), t, V, eps)
    S = _Sector(nx, ny, c["px"], c["py"], c["U"], t, V, eps)
    if c["op"] == "sector_h":
        return S.ham(_vector(c, seed, S.D.numel()).reshape(S.D.shape)).flatten()
    theta = _angles(rng, L * S.per)
    if c["op"] == "ansatz":
        psi = S.forward(theta)
        full = torch.zeros(1 << (2 * ns), dtype=torch.complex128, device=S.dev)
        at = (torch.tensor(S.pats[1], device=S.dev)[:, None] << ns) + torch.tensor(
            S.pats[0], device=S.dev)[None, :]
        full[at.flatten()] = psi.flatten()
        return full
    return S.grad(theta)
