"""Performance cases of the exact-diagonalisation library: what they are, the
work each stands for, and plain reference values for them.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)`
further ones of the same ranges, `prepare(case, seed)` what a program holds
before the call (model, basis, plan, vectors), `run(state)` one pass through
the public entry points, `work(case)` the bytes and operations of a pass, and
`exact(case, seed)` the same outputs from plain FP64 torch and numpy.

Kinds:
  hv       H.v through a plan, nvec vectors (the inner product of everything else)
  lanczos  a fixed number of Lanczos steps, coefficients only
  gs       a converged Lanczos ground state with its vector
  cf       continued-fraction Green function from a given state
  batch    many small impurity solves (ground state and 4x4 Green function) at once
  cdmft    one CDMFT iteration: impurity solve, Green function, lattice average, bath fit
  vca      one value of the Potthoff functional: reference solve, band Lanczos, k sum
  sym      the stored-matrix product in a symmetry-adapted sector
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_2305_18643_amd as q

DEV = "cuda"


# ---------------------------------------------------------------- models

def _bonds_of(geom, L):
    """Nearest-neighbour pairs and plaquette diagonals of a geometry."""
    if geom == "chain":
        nx, ny = L, 1
    elif geom == "ladder":
        nx, ny = L // 2, 2
    else:
        nx, ny = {4: (2, 2), 9: (3, 3), 12: (4, 3), 16: (4, 4)}[L]
    nn, diag = [], []
    for y, x in itertools.product(range(ny), range(nx)):
        a = x + nx * y
        if x + 1 < nx:
            nn.append((a, a + 1))
        if y + 1 < ny:
            nn.append((a, a + nx))
        if x + 1 < nx and y + 1 < ny:
            diag += [(a, a + nx + 1), (a + 1, a + nx)]
    return nn, diag, nx, ny


def _lattice(geom, L, U, t=-1.0, tp=0.0, spread=0.0, rng=None):
    """t = -1 (with a spread per bond, as the serving requests have) on the
    nearest neighbours, tp on the diagonals, mu = U/2."""
    T = np.zeros((L, L))
    nn, diag, _, _ = _bonds_of(geom, L)
    for a, b in nn:
        T[a, b] = T[b, a] = t + (spread * rng.standard_normal() if spread else 0.0)
    for a, b in diag:
        if tp:
            T[a, b] = T[b, a] = tp
    T[np.diag_indices(L)] = -U / 2
    return T, np.full(L, float(U))


def _impurity(rng, n_bath):
    """A 2x2 plaquette with n_bath bath orbitals (the batched workload)."""
    n = 4 + n_bath
    T = np.zeros((n, n))
    for a, b in ((0, 1), (2, 3), (0, 2), (1, 3)):
        T[a, b] = T[b, a] = -1.0
    U = rng.uniform(2.0, 10.0)
    T[np.arange(4), np.arange(4)] = -U / 2
    for a in range(n_bath):
        T[4 + a, a % 4] = T[a % 4, 4 + a] = rng.uniform(0.2, 1.0)
        T[4 + a, 4 + a] = rng.uniform(-3.0, 3.0)
    Us = np.zeros(n)
    Us[:4] = U
    return T, Us, int(rng.choice([n // 2, (n + 1) // 2])), int(rng.choice([n // 2, (n + 1) // 2]))


def _model(case, seed):
    """(t, U) of a single-model case; the seed moves U a little, so that other
    seeds are other Hamiltonians of the same kind."""
    rng = np.random.default_rng([seed, 1])
    U = case["U"] + rng.uniform(-0.1, 0.1)
    if case["geom"] == "impurity":
        T, Us, _, _ = _impurity(rng, case["L"] - 4)
        return T, Us
    return _lattice(case["geom"], case["L"], U, tp=case.get("tp", 0.0),
                    spread=case.get("spread", 0.0), rng=rng)


def _vector(n, seed, dtype=torch.float64):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + 17)
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64).mul_(2).sub_(1).to(dtype)


# ---------------------------------------------------------------- plain FP64 reference

class _Spin:
    """Strings of one spin in ascending order and, per bond, the signed hop."""

    def __init__(self, T, L, N):
        s = [sum(1 << k for k in c) for c in itertools.combinations(range(L), N)]
        self.s = np.array(sorted(s), dtype=np.int64)
        self.d = len(s)
        self.e = sum(((self.s >> k) & 1) * T[k, k] for k in range(L)) + np.zeros(self.d)
        self.col, self.coef = [], []
        for a in range(L):
            for b in range(a + 1, L):
                if T[a, b] == 0.0:
                    continue
                oa, ob = (self.s >> a) & 1, (self.s >> b) & 1
                ok = oa != ob
                y = np.where(ok, self.s ^ ((1 << a) | (1 << b)), self.s)
                between = ((1 << b) - 1) & ~((1 << (a + 1)) - 1)
                m = _popcount(self.s & between) & 1
                self.col.append(torch.from_numpy(np.searchsorted(self.s, y)).to(DEV))
                self.coef.append(torch.from_numpy(np.where(ok, T[a, b] * (1.0 - 2.0 * m), 0.0)).to(DEV))


def _popcount(x):
    x = np.asarray(x, dtype=np.int64)
    n = np.zeros_like(x)
    while x.any():
        n += x & 1
        x = x >> 1
    return n


class _Ham:
    """H of one sector as V K_up^T + K_dn V + D o V, V[i_dn, i_up], in torch."""

    def __init__(self, T, U, nup, ndn):
        L = T.shape[0]
        self.up, self.dn = _Spin(T, L, nup), _Spin(T, L, ndn)
        self.dim = self.up.d * self.dn.d
        self.diag = (torch.from_numpy(self.dn.e).to(DEV)[:, None] + torch.from_numpy(self.up.e).to(DEV)[None, :])
        for k in range(L):
            if U[k]:
                nu = torch.from_numpy((self.up.s >> k & 1).astype(np.float64)).to(DEV)
                nd = torch.from_numpy((self.dn.s >> k & 1).astype(np.float64)).to(DEV)
                self.diag.addcmul_(nd[:, None], nu[None, :], value=float(U[k]))

    def __call__(self, v):
        """H v for one flat vector or a batch [n, dim]."""
        V = v.reshape(-1, self.dn.d, self.up.d)
        W = V * self.diag
        for col, c in zip(self.up.col, self.up.coef):
            W.addcmul_(V.index_select(2, col), c[None, None, :])
        for col, c in zip(self.dn.col, self.dn.coef):
            W.addcmul_(V.index_select(1, col), c[None, :, None])
        return W.reshape(v.shape)

    def dense(self):
        return self(torch.eye(self.dim, dtype=torch.float64, device=DEV))


def _lanczos(H, v0, steps, tol=0.0, keep=False):
    """Plain Lanczos from v0; keep: every vector kept and reorthogonalised
    against, and the lowest Ritz pair, stopped at the residual tol."""
    v = v0 / v0.norm()
    vp, a, b, vs, brk = None, [], [], [], False
    for n in range(steps):
        if keep:
            vs.append(v)
        w = H(v)
        if vp is not None:
            w -= b[-1] * vp
        a.append(float(torch.dot(v, w)))
        w -= a[-1] * v
        if keep:
            for _ in range(2):
                for u in vs:
                    w -= torch.dot(u, w) * u
        b.append(float(w.norm()))
        if keep and (n % 4 == 3 or n + 1 == steps or b[-1] < 1e-10):
            T = np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1)
            th, s = np.linalg.eigh(T)
            if abs(b[-1] * s[-1, 0]) <= tol * max(1.0, abs(th[0])) or b[-1] < 1e-10:
                break
        vp, v = v, w / b[-1]
    if not keep:
        return np.array(a), np.array(b)
    s0 = s[:, 0] * (1.0 if s[0, 0] >= 0 else -1.0)
    psi = torch.zeros_like(v0)
    for c, u in zip(s0, vs):
        psi += float(c) * u
    return float(th[0]), psi / psi.norm()


def _ladder_up(T, psi, src, tgt, ops, create):
    """sum over ops of c+_o (or c_o) psi on the up strings: src -> tgt tables."""
    out = torch.zeros(psi.shape[0], tgt.d, dtype=torch.float64, device=DEV)
    for o in ops:
        bit = 1 << o
        ok = ((tgt.s & bit) != 0) == create
        below = _popcount(tgt.s & (bit - 1)) & 1
        col = np.searchsorted(src.s, np.where(ok, tgt.s ^ bit, src.s[0]))
        c = np.where(ok, 1.0 - 2.0 * below, 0.0)
        out.addcmul_(psi.index_select(1, torch.from_numpy(col).to(DEV)), torch.from_numpy(c).to(DEV)[None, :])
    return out


# ---------------------------------------------------------------- per kind

def _grid(n=64):
    return -10.0 + 20.0 * np.arange(n) / (n - 1) + 0.1j


def _jobs(case, seed):
    """The impurity models of a batch: bath sizes spread evenly over the range."""
    rng = np.random.default_rng([seed, 2])
    lo, hi, n = case["bath_lo"], case["bath_hi"], case["jobs"]
    return [_impurity(rng, lo + (hi - lo) * k // max(n - 1, 1)) for k in range(n)]


class _Cdmft:
    """The 1D chain on 4-site clusters with 4 bath orbitals at energies eb1, eb2."""

    def __init__(self, case, seed):
        rng = np.random.default_rng([seed, 3])
        L, nb = 4, 4
        self.U = case["U"] + rng.uniform(-0.1, 0.1)
        self.mu = self.U / 2
        self.tc = np.zeros((L, L))
        for i in range(L - 1):
            self.tc[i, i + 1] = self.tc[i + 1, i] = -1.0
        self.A_eps = np.zeros((nb, 4))
        self.A_eps[0, 0] = self.A_eps[1, 0] = self.A_eps[2, 1] = self.A_eps[3, 1] = 1.0
        self.A_theta = np.zeros((L * nb, 4))
        self.A_theta[[0, 3 * nb + 1], 2] = -1.0
        self.A_theta[[2, 3 * nb + 3], 3] = -1.0
        self.nup = self.ndn = 4
        self.bonds = [(3, 0, (1, 0, 0), -1.0)]
        e, th = rng.uniform(0.9, 1.3), rng.uniform(0.6, 1.0)
        self.p0 = np.array([e, -e, th, th])
        n = np.arange(int((case["wc"] * case["beta"] / math.pi - 1.0) / 2.0) + 1)
        self.z = 1j * (2 * n + 1) * math.pi / case["beta"]
        self.w = np.full(len(self.z), 1.0 / len(self.z))
        self.ks = np.stack([np.arange(case["nk"]) / case["nk"], np.zeros(case["nk"]), np.zeros(case["nk"])], axis=1)


class _Vca:
    """The square lattice tiled by plaquettes; the reference's hopping tp is the
    variational parameter."""

    def __init__(self, case, seed):
        rng = np.random.default_rng([seed, 4])
        U = case["U"] + rng.uniform(-0.1, 0.1)
        tp = case["tp"] + rng.uniform(-0.02, 0.02)
        self.t_ref, self.U = _lattice("rect", 4, U, t=tp)
        self.nup = self.ndn = 2
        self.dt = _lattice("rect", 4, U, t=-1.0)[0] - self.t_ref
        self.bonds = [(1, 0, (1, 0, 0), -1.0), (3, 2, (1, 0, 0), -1.0), (2, 0, (0, 1, 0), -1.0), (3, 1, (0, 1, 0), -1.0)]
        n = case["nk"]
        m, l = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
        self.ks = np.stack([m.ravel() / n, l.ravel() / n, np.zeros(n * n)], axis=1)


def _group(case):
    """(permutations, characters): the mirror of a chain, or C2v of a rectangle."""
    _, _, nx, ny = _bonds_of(case["geom"], case["L"])
    site = lambda x, y: x + nx * y  # noqa: E731
    xy = [(a % nx, a // nx) for a in range(nx * ny)]
    if ny == 1:
        return [list(range(nx)), [nx - 1 - x for x, _ in xy]], [1, case["chi"][0]]
    cx, cy = case["chi"][0], case["chi"][1]
    return ([list(range(nx * ny)), [site(nx - 1 - x, ny - 1 - y) for x, y in xy],
             [site(x, ny - 1 - y) for x, y in xy], [site(nx - 1 - x, y) for x, y in xy]],
            [1, cx * cy, cy, cx])


def _sym_case(case):
    perms, chi = _group(dict(case, chi=[int(c) for c in (case["chi_x"], case["chi_y"])]))
    return perms, chi


def _dim(L, nup, ndn):
    return math.comb(L, nup) * math.comb(L, ndn)


def _sym_dim(case):
    return _dim(case["L"], case["nup"], case["ndn"]) // len(_sym_case(case)[0])


# ---------------------------------------------------------------- the interface

def listed():
    return [
        # the smallest product there is: the 2x2 plaquette, one launch's latency
        dict(name="hv_plaquette", kind="hv", geom="rect", L=4, nup=2, ndn=2, U=8.0, prec="fp64", nvec=1),
        # a 10-orbital impurity's product over the 10 chains of a 4x4 Green function,
        # FP32 vectors, every bond another amplitude
        dict(name="hv_impurity10_x10", kind="hv", geom="impurity", L=10, nup=5, ndn=5, U=4.0, prec="fp32v", nvec=10),
        # the 14-site chain, the largest sector of the batched and served solves
        dict(name="hv_chain14", kind="hv", geom="chain", L=14, nup=7, ndn=7, U=4.0, prec="fp64", nvec=1),
        # the 4x4 cluster at half filling: the headline product, in both storage types
        dict(name="hv_4x4_fp64", kind="hv", geom="rect", L=16, nup=8, ndn=8, U=8.0, prec="fp64", nvec=1),
        dict(name="hv_4x4_fp32v", kind="hv", geom="rect", L=16, nup=8, ndn=8, U=8.0, prec="fp32v", nvec=1),
        # Lanczos steps on the 4x4 cluster (a ground state there takes 200 to 300 of them)
        dict(name="lanczos_4x4", kind="lanczos", geom="rect", L=16, nup=8, ndn=8, U=8.0, prec="fp64", steps=8),
        # a whole converged ground state of a served request's size (12 orbitals)
        dict(name="gs_ladder12", kind="gs", geom="ladder", L=12, nup=6, ndn=6, U=6.0, spread=0.2, prec="fp64"),
        # the continued-fraction Green function of the 14-site chain: 4 orbitals,
        # 10 pairs x 2 parts run together
        dict(name="cf_chain14", kind="cf", geom="chain", L=14, nup=7, ndn=7, U=4.0, norb=4, floors=12),
        # a batch of impurity solves as CDMFT and VCA runs hand them over: 6 to 12
        # orbitals, FP32 vectors, 100-floor Green functions
        dict(name="batch_24", kind="batch", jobs=24, bath_lo=2, bath_hi=8, prec="fp32v", floors=100),
        # one iteration of the CDMFT loop of the 1D model (4 sites, 4 bath orbitals)
        dict(name="cdmft_iteration", kind="cdmft", U=4.0, beta=50.0, wc=2.0, nk=64, floors=200),
        # one value of the Potthoff functional on a 32 x 32 grid (a VCA scan asks for many)
        dict(name="vca_plaquette", kind="vca", U=8.0, tp=-1.0, nk=32, method="poles"),
        # the stored-matrix product of the 4x4 cluster's A1 sector, packed
        dict(name="sym_4x4_a1", kind="sym", geom="rect", L=16, nup=8, ndn=8, U=8.0, chi_x=1, chi_y=1, packed=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_hv(rng):
    while True:
        L = rng.randint(4, 15)
        geom = rng.choice(["chain", "impurity", "ladder" if L % 2 == 0 else "chain", "rect" if L in (4, 9, 12) else "impurity"])
        if geom == "impurity" and L < 6:
            continue
        c = dict(kind="hv", geom=geom, L=L, nup=max(1, L // 2 - rng.randint(0, 2)), ndn=max(1, (L + 1) // 2 - rng.randint(0, 2)),
                 U=round(rng.uniform(2.0, 10.0), 4), prec=rng.choice(["fp64", "fp32v"]), nvec=_log_int(rng, 1, 20))
        if geom == "rect":
            c["tp"] = rng.choice([0.0, 0.3])
        if c["nvec"] * _dim(L, c["nup"], c["ndn"]) <= 120_000_000:
            return c


def draw(rng):
    kind = rng.choice(["hv", "hv", "hv", "gs", "cf", "batch", "cdmft", "vca", "sym"])
    U = round(rng.uniform(2.0, 10.0), 4)
    if kind == "hv":
        return _draw_hv(rng)
    if kind == "gs":
        L = rng.randint(6, 13)
        return dict(kind="gs", geom="ladder" if L % 2 == 0 and rng.random() < 0.5 else "chain", L=L, nup=(L + 1) // 2,
                    ndn=L // 2, U=U, spread=0.2, prec="fp64")
    if kind == "cf":
        L = rng.randint(8, 13)
        return dict(kind="cf", geom="chain", L=L, nup=(L + 1) // 2, ndn=L // 2, U=U, norb=rng.randint(1, 4), floors=rng.randint(8, 12))
    if kind == "batch":
        lo = rng.randint(2, 5)
        return dict(kind="batch", jobs=rng.randint(3, 20), bath_lo=lo, bath_hi=rng.randint(lo, 8), prec=rng.choice(["fp32v", "fp64"]),
                    floors=rng.randint(20, 100))
    if kind == "cdmft":
        return dict(kind="cdmft", U=round(rng.uniform(2.0, 6.0), 4), beta=float(rng.randint(30, 60)), wc=2.0, nk=_log_int(rng, 16, 128), floors=200)
    if kind == "vca":
        return dict(kind="vca", U=round(rng.uniform(4.0, 10.0), 4), tp=round(-rng.uniform(0.6, 1.4), 4),
                    nk=_log_int(rng, 8, 32), method=rng.choice(["poles", "quad"]))
    geom, L = rng.choice([("chain", 10), ("chain", 12), ("chain", 13), ("chain", 14), ("rect", 12)])
    return dict(kind="sym", geom=geom, L=L, nup=L // 2 - rng.randint(0, 1), ndn=L // 2 - rng.randint(0, 1), U=U,
                chi_x=rng.choice([1, -1]), chi_y=rng.choice([1, -1]), packed=rng.random() < 0.5)


def prepare(case, seed):
    k = case["kind"]
    st = dict(case=case)
    if k == "batch":
        st["specs"] = [q.JobSpec((T, U), nup, ndn, orbs=range(4), seed=j + 1) for j, (T, U, nup, ndn) in enumerate(_jobs(case, seed))]
        st["z"] = _grid()
        return st
    if k == "cdmft":
        st["prob"] = _Cdmft(case, seed)
        return st
    if k == "vca":
        st["prob"] = _Vca(case, seed)
        return st
    T, U = _model(case, seed)
    st["model"] = m = q.HostModel(T, U)
    st["basis"] = b = q.sector_basis(case["L"], case["nup"], case["ndn"])
    if k == "hv":
        dt = torch.float64 if case["prec"] == "fp64" else torch.float32
        st["plan"] = q.HvPlan(m, b, case["prec"])
        st["v"] = _vector(case["nvec"] * b.dim, seed, dt)
        st["w"] = torch.empty_like(st["v"])
    elif k in ("lanczos", "gs"):
        st["v0"] = _vector(b.dim, seed)
    elif k == "cf":
        H = _Ham(T, U, case["nup"], case["ndn"])
        st["e0"], st["psi"] = _lanczos(H, _vector(b.dim, seed), 30, keep=True)
    elif k == "sym":
        perms, chi = _sym_case(case)
        sec = q.sym_sector(b, perms, chi)
        st["H"] = H = q.sym_hamiltonian(m, sec)
        if case["packed"]:
            H.pack()
        st["v"] = _vector(H.dim, seed)
        st["w"] = torch.empty_like(st["v"])
    return st


def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "hv":
        return st["plan"](st["v"], st["w"], case["nvec"])
    if k == "lanczos":
        r = q.lanczos_gs(st["model"], st["basis"], fixed_steps=case["steps"], want_vector=False, check_every=case["steps"],
                         prec=case["prec"], v0=st["v0"])
        return dict(alpha=r["alpha"], beta=r["beta"], e0=np.array([r["e0"]]))
    if k == "gs":
        r = q.lanczos_gs(st["model"], st["basis"], prec=case["prec"], v0=st["v0"])
        return dict(e0=np.array([r["e0"]]), psi=r["psi"])
    if k == "cf":
        r = q.green_cf(st["model"], st["basis"], st["psi"], st["e0"], range(case["norb"]), _grid(), max_steps=case["floors"])
        return dict(G=r["G"], coef=r["coef"])
    if k == "batch":
        rs = q.batch_solve(st["specs"], prec=case["prec"], gf_steps=case["floors"], z=st["z"])
        return dict(e0=np.array([r["e0"] for r in rs]), G=np.stack([r["G"] for r in rs]))
    if k == "cdmft":
        p = st["prob"]
        r = q.cdmft(p, p.p0, p.ks, p.z, p.w, max_iter=1, max_steps=case["floors"])
        return dict(p=r["p"], e0=np.array([r["e0"]]), Gc=r["Gc"], sigma=r["sigma"], gbar=r["gbar"], g0inv=r["g0inv"])
    if k == "vca":
        p = st["prob"]
        return np.array([q.vca.omega(p, p.ks, method=case["method"])])
    return st["H"](st["v"], st["w"])


def work(case):
    """Bytes and FP64 operations of a pass.  Per vector element a product reads
    v and writes w and does a multiply-add for the diagonal and for each hop; a
    Lanczos step reads v_n and v_{n-1} and writes v_{n+1}."""
    k = case["kind"]
    if k in ("hv", "lanczos", "gs", "cf"):
        L, s = case["L"], 8 if case.get("prec", "fp64") == "fp64" else 4
        if case["geom"] == "impurity":
            nb = L
        else:
            nn, diag, _, _ = _bonds_of(case["geom"], L)
            nb = len(nn) + (len(diag) if case.get("tp") else 0)

        def ops(nup, ndn):
            hops = sum(2.0 * n * (L - n) / (L * (L - 1)) * nb for n in (nup, ndn))
            return 2.0 * (1 + hops) * _dim(L, nup, ndn)
        d, f = _dim(L, case["nup"], case["ndn"]), ops(case["nup"], case["ndn"])
        if k == "hv":
            return dict(bytes=2 * s * d * case["nvec"], flops=f * case["nvec"])
        if k == "lanczos":
            return dict(bytes=3 * s * d * case["steps"], flops=(f + 10 * d) * case["steps"])
        if k == "gs":   # about 8 L steps to the residual test
            return dict(bytes=3 * s * d * 8 * L, flops=(f + 10 * d) * 8 * L)
        pairs = case["norb"] * (case["norb"] + 1) // 2
        both = [(case["nup"] + 1, case["ndn"]), (case["nup"] - 1, case["ndn"])]
        n = pairs * case["floors"]
        return dict(bytes=n * sum(3 * s * _dim(L, *p) for p in both), flops=n * sum(ops(*p) + 10 * _dim(L, *p) for p in both))
    if k == "batch":
        s, by, fl = 8 if case["prec"] == "fp64" else 4, 0.0, 0.0
        lo, hi, n = case["bath_lo"], case["bath_hi"], case["jobs"]
        for j in range(n):
            L = 4 + lo + (hi - lo) * j // max(n - 1, 1)
            d = _dim(L, L // 2, L // 2)
            steps = 60 + 20 * case["floors"]
            by += 3 * s * d * steps
            fl += (2.0 * (1 + 0.55 * 2 * L) + 10) * d * steps
        return dict(bytes=by, flops=fl)
    if k == "cdmft":
        d, steps = _dim(8, 4, 4), 80 + 20 * case["floors"]
        return dict(bytes=3 * 8 * d * steps, flops=30.0 * d * steps)
    if k == "vca":
        nk, R = case["nk"] ** 2, 24
        return dict(bytes=nk * 24.0 + 36 * 8 * 3 * 30, flops=nk * 4.0 / 3 * 8 * R ** 3)
    d = _sym_dim(case)
    nn, _, _, _ = _bonds_of(case["geom"], case["L"])
    L = case["L"]
    nnz = d * (1 + sum(2.0 * n * (L - n) / (L * (L - 1)) * len(nn) for n in (case["nup"], case["ndn"])))
    return dict(bytes=nnz * (4 if case["packed"] else 12) + 24.0 * d, flops=2.0 * nnz)


# ---------------------------------------------------------------- reference values

def _exact_sym(case, seed):
    """w = B^T H B v with the isometry B from the symmetry-adapted to the full
    sector: each kept orbit's smallest label represents it."""
    T, U = _model(case, seed)
    perms, chi = _sym_case(case)
    L = case["L"]
    H = _Ham(T, U, case["nup"], case["ndn"])

    def images(sp):
        lab, sg = [], []
        for p in perms:
            y, par = np.zeros_like(sp.s), np.zeros_like(sp.s)
            for a in range(L):
                y |= ((sp.s >> a) & 1) << p[a]
                for b in range(a + 1, L):
                    if p[a] > p[b]:
                        par ^= (sp.s >> a) & (sp.s >> b) & 1
            lab.append(torch.from_numpy(np.searchsorted(sp.s, y)).to(DEV))
            sg.append(torch.from_numpy(1.0 - 2.0 * par).to(DEV))
        return lab, sg
    lu, su = images(H.up)
    ld, sd = images(H.dn)
    own = torch.arange(H.dim, device=DEV)
    low, phase, stab = own.clone(), torch.ones(H.dim, dtype=torch.float64, device=DEV), torch.zeros(H.dim, dtype=torch.float64, device=DEV)
    for g in range(len(perms)):
        lab = (lu[g][None, :] + H.up.d * ld[g][:, None]).reshape(-1)
        sg = (sd[g][:, None] * su[g][None, :]).reshape(-1) * chi[g]
        stab += torch.where(lab == own, sg, 0.0)
        less = lab < low
        low = torch.where(less, lab, low)
        phase = torch.where(less, sg, phase)
        del lab, sg, less
    keep = stab > 0.5
    rep = torch.nonzero((low == own) & keep).reshape(-1)
    idx = torch.searchsorted(rep, low).clamp_(max=rep.numel() - 1)
    # an orbit of n_g / stab states, each with amplitude phase * sqrt(stab / n_g)
    amp = torch.where(keep, phase * torch.sqrt(stab.clamp(min=0.0) / len(perms)), 0.0)
    del low, phase, stab, own, keep
    full = _vector(rep.numel(), seed)[idx] * amp
    return torch.zeros(rep.numel(), dtype=torch.float64, device=DEV).index_add_(0, idx, H(full) * amp)


def _exact_cf(case, seed):
    T, U = _model(case, seed)
    H = _Ham(T, U, case["nup"], case["ndn"])
    e0, psi = _lanczos(H, _vector(H.dim, seed), 30, keep=True)
    psi = psi.reshape(H.dn.d, H.up.d)
    n, M, z = case["norb"], case["floors"], _grid()
    pairs = [(i, j) for i in range(n) for j in range(i, n)]
    coef = np.zeros((len(pairs), 2, 1 + 2 * M))
    F = np.zeros((len(pairs), len(z)), dtype=complex)
    for part, nup in enumerate((case["nup"] + 1, case["nup"] - 1)):
        Hp = _Ham(T, U, nup, case["ndn"])
        sg = 1.0 if part == 0 else -1.0
        for p, (i, j) in enumerate(pairs):
            phi = _ladder_up(T, psi, H.up, Hp.up, (i,) if i == j else (i, j), part == 0).reshape(-1)
            b0 = float(torch.dot(phi, phi))
            a, b = _lanczos(Hp, phi, M)
            coef[p, part, 0], coef[p, part, 1:1 + M], coef[p, part, 1 + M:2 * M] = b0, a, b[:-1] ** 2
            g = z + sg * e0 - sg * a[-1]
            for f in range(M - 2, -1, -1):
                g = z + sg * e0 - sg * a[f] - b[f] ** 2 / g
            F[p] += b0 / g
    G = np.zeros((len(z), n, n), dtype=complex)
    at = {pr: k for k, pr in enumerate(pairs)}
    for (i, j), k in at.items():
        G[:, i, j] = G[:, j, i] = F[k] if i == j else 0.5 * (F[k] - F[at[i, i]] - F[at[j, j]])
    return dict(G=G, coef=coef)


def _exact_cdmft(case, seed):
    p = _Cdmft(case, seed)
    L, nb = 4, 4
    eps, th = p.A_eps @ p.p0, (p.A_theta @ p.p0).reshape(L, nb)
    tcp = p.tc - p.mu * np.eye(L)
    T = np.block([[tcp, th], [th.T, np.diag(eps)]])
    U = np.array([p.U] * L + [0.0] * nb)
    H = _Ham(T, U, 4, 4)
    e0, psi = _lanczos(H, _vector(H.dim, 1), 300, tol=1e-13, keep=True)
    psi = psi.reshape(H.dn.d, H.up.d)
    G = np.zeros((len(p.z), L, L), dtype=complex)
    for part, nup in enumerate((5, 3)):
        Hp = _Ham(T, U, nup, 4)
        sg = 1.0 if part == 0 else -1.0
        phi = torch.stack([_ladder_up(T, psi, H.up, Hp.up, (i,), part == 0).reshape(-1) for i in range(L)])
        D = Hp.dense().to(torch.complex128)
        for k, z in enumerate(p.z):
            A = -sg * D
            A.diagonal().add_(complex(z) + sg * e0)
            x = torch.linalg.solve(A, phi.to(torch.complex128).T)
            G[k] += (phi.to(torch.complex128) @ x).cpu().numpy()
    one = np.eye(L)
    sigma, gbar, g0 = (np.zeros_like(G) for _ in range(3))
    for k, z in enumerate(p.z):
        sigma[k] = z * one - tcp - (th / (z - eps)) @ th.T - np.linalg.inv(G[k])
        for kk in p.ks:
            V = np.zeros((L, L), dtype=complex)
            for i, j, sh, t in p.bonds:
                ph = t * np.exp(2j * math.pi * float(np.dot(kk, sh)))
                V[i, j] += ph
                V[j, i] += np.conj(ph)
            gbar[k] += np.linalg.inv(z * one - tcp - V - sigma[k]) / len(p.ks)
        g0[k] = np.linalg.inv(gbar[k]) + sigma[k]
    return dict(p=None, e0=np.array([e0]), Gc=G, sigma=sigma, gbar=gbar, g0inv=g0)


def _exact_vca(case, seed):
    p = _Vca(case, seed)
    H = _Ham(p.t_ref, p.U, 2, 2)
    th, S = np.linalg.eigh(H.dense().cpu().numpy())
    e0, psi = th[0], torch.from_numpy(S[:, 0].copy()).to(DEV).reshape(H.dn.d, H.up.d)
    poles, Q = [], []
    for part, nup in enumerate((3, 1)):
        Hp = _Ham(p.t_ref, p.U, nup, 2)
        lam, V = np.linalg.eigh(Hp.dense().cpu().numpy())
        phi = np.stack([_ladder_up(p.t_ref, psi, H.up, Hp.up, (i,), part == 0).reshape(-1).cpu().numpy() for i in range(4)])
        c = phi @ V
        poles.append(lam - e0 if part == 0 else e0 - lam)
        Q.append(c)
    poles, Q = np.concatenate(poles), np.concatenate(Q, axis=1)
    tot = 0.0
    for kk in p.ks:
        V = p.dt.astype(complex)
        for i, j, sh, t in p.bonds:
            ph = t * np.exp(2j * math.pi * float(np.dot(kk, sh)))
            V[i, j] += ph
            V[j, i] += np.conj(ph)
        w = np.linalg.eigvalsh(np.diag(poles) + Q.T @ V @ Q)
        tot += w[w < 0].sum()
    return np.array([e0 + 2.0 * (tot / len(p.ks) - poles[poles < 0].sum())])


def exact(case, seed):
    k = case["kind"]
    if k == "batch":
        e = []
        for T, U, nup, ndn in _jobs(case, seed):
            H = _Ham(T, U, nup, ndn)
            e.append(_lanczos(H, _vector(H.dim, 1), 240, tol=1e-10, keep=True)[0])
        return dict(e0=np.array(e), G=None)
    if k == "cdmft":
        return _exact_cdmft(case, seed)
    if k == "vca":
        return _exact_vca(case, seed)
    if k == "sym":
        return _exact_sym(case, seed)
    if k == "cf":
        return _exact_cf(case, seed)
    T, U = _model(case, seed)
    H = _Ham(T, U, case["nup"], case["ndn"])
    if k == "hv":
        v = _vector(case["nvec"] * H.dim, seed, torch.float64 if case["prec"] == "fp64" else torch.float32).double()
        if case["nvec"] * H.dim < 20_000_000:
            return H(v.reshape(case["nvec"], H.dim)).reshape(-1)
        return torch.cat([H(x) for x in v.reshape(case["nvec"], H.dim)])
    if k == "lanczos":
        a, b = _lanczos(H, _vector(H.dim, seed), case["steps"])
        th = np.linalg.eigvalsh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
        return dict(alpha=a, beta=b, e0=th[:1])
    e0, psi = _lanczos(H, _vector(H.dim, seed), 400, tol=1e-13, keep=True)
    return dict(e0=np.array([e0]), psi=psi)
