"""The fused product and its Lanczos step at the edges of the kernel's tiling:
rows of one string, a few strings, a row past a tile of 64 or 128 strings, odd
rows per block and odd rows left over, one row per block with odd lengths, rows
whose pair does not fit LDS, hop counts past the sixteen that are read ahead,
and vectors whose byte offsets leave 31 bits.

Tolerance of a product: the rounding of a sum of n terms, (n + 2) eps (|H||v|)_i
with n = 2 bonds + 1, and for FP32 vectors one rounding of the result.  The
coefficients of the first Lanczos steps: 1e-12 relative to |H| in FP64."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    q.load_library()
    return q


def _models():
    out = [synth.random_model(701, 10, 0, 5), synth.random_model(702, 10, 10, 3),   # d_up = 1
           synth.random_model(703, 3, 1, 2), synth.random_model(704, 2, 1, 1),      # d_up = 3, 2
           synth.random_model(705, 1, 1, 0),
           synth.random_model(706, 8, 4, 3),                   # 70 strings, 29 rows per block
           synth.random_model(707, 12, 2, 5, uniform_U=True),  # 66 strings, 31 rows per block
           synth.chain(9, U=4.0, mu=2.0, nup=4, ndn=5),        # 126 strings, one t
           synth.random_model(708, 12, 6, 1, density=1.0),     # 66 bonds, up to 36 hops
           synth.random_model(709, 20, 3, 1, density=0.2),     # one row per block, 1140 strings
           synth.random_model(710, 23, 3, 1, density=0.2),     # 1771 strings, 23 rows
           synth.chain(23, U=3.0, mu=1.5, nup=3, ndn=22),      # one t, odd rows
           synth.chain(27, U=2.0, mu=1.0, nup=4, ndn=1)]       # 17550 strings
    return out


@pytest.mark.parametrize("m", _models(), ids=lambda m: f"{m.name}_{m.nup}_{m.ndn}")
@pytest.mark.parametrize("prec", ["fp64", "fp32v"])
@pytest.mark.parametrize("nvec", [1, 3])
def test_product(q, m, prec, nvec):
    import torch
    print(f"product {m.name} ({m.nup},{m.ndn}) {prec} x{nvec}", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    dt = torch.float64 if prec == "fp64" else torch.float32
    v = np.random.default_rng(11).uniform(-1, 1, (nvec, b.dim))
    v = torch.tensor(v, dtype=dt)
    plan = q.HvPlan(m, b, prec)
    # a vector of its own before and after: nothing outside w is written
    buf = torch.full((nvec * b.dim + 256,), 7.5, dtype=dt, device="cuda")
    w = buf[128:128 + nvec * b.dim]
    plan(v.cuda().reshape(-1), w, nvec)
    assert bool((buf[:128] == 7.5).all()) and bool((buf[128 + nvec * b.dim:] == 7.5).all())
    got = w.double().cpu().numpy().reshape(nvec, b.dim)
    terms = 2 * int(np.count_nonzero(np.triu(m.t, 1))) + 3
    for k in range(nvec):
        x = v[k].double().numpy()
        ref = oracle.hv(m.t, m.U, m.nup, m.ndn, x)
        bound = oracle.hv_abs_bound(m.t, m.U, m.nup, m.ndn, x)
        tol = (terms + 2) * EPS * bound + 1e-300
        if prec == "fp32v":
            tol = tol + 2.0 ** -24 * np.abs(ref) * (1 + 2.0 ** -20)
        assert np.all(np.abs(got[k] - ref) <= tol)


@pytest.mark.parametrize("m", [m for m in _models() if oracle.binom(m.L, m.nup) * oracle.binom(m.L, m.ndn) > 60],
                         ids=lambda m: f"{m.name}_{m.nup}_{m.ndn}")
def test_first_lanczos_steps(q, m):
    import torch
    print(f"steps {m.name} ({m.nup},{m.ndn})", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    x = np.random.default_rng(12).uniform(-1, 1, b.dim)
    r = q.lanczos_gs(m, b, fixed_steps=4, want_vector=False, v0=torch.tensor(x, device="cuda"))
    v, vp, beta = x / np.linalg.norm(x), None, 0.0
    scale = np.abs(m.t).sum() + m.U.sum()
    for n in range(4):
        w = oracle.hv(m.t, m.U, m.nup, m.ndn, v)
        if n:
            w = w - beta * vp
        alpha = float(v @ w)
        w = w - alpha * v
        beta = float(np.linalg.norm(w))
        assert abs(r["alpha"][n] - alpha) <= 1e-12 * scale, (n, r["alpha"][n], alpha)
        assert abs(r["beta"][n] - beta) <= 1e-12 * scale, (n, r["beta"][n], beta)
        v, vp = w / beta, v


@pytest.mark.parametrize("L,nup,ndn", [(24, 2, 9), (23, 3, 7)])
def test_product_over_2gb_sampled_rows(q, L, nup, ndn):
    """FP64 vectors of 2.9 GB (276 strings a row) and 3.5 GB (1771): neighbour
    rows through 64-bit addresses; oracle rows computed one by one."""
    import torch
    m = synth.random_model(720, L, nup, ndn, density=0.15)
    print(f"product {L} orbitals ({nup},{ndn})", flush=True)
    b = q.sector_basis(L, nup, ndn)
    assert b.dim * 8 > 2 ** 31
    v = oracle.start_vector(7, b.dim)
    rows = np.unique(np.concatenate([np.random.default_rng(13).integers(0, b.dim, 2000), np.arange(64),
                                     np.arange(b.dim - 64, b.dim)]))
    w = q.hv(m, b, torch.from_numpy(v).cuda())
    got = w[torch.from_numpy(rows).cuda()].cpu().numpy()
    del w
    ref = oracle.hv_rows(m.t, m.U, nup, ndn, v, rows)
    bound = oracle.hv_abs_bound(m.t, m.U, nup, ndn, v, rows)
    terms = 2 * int(np.count_nonzero(np.triu(m.t, 1))) + 3
    assert np.all(np.abs(got - ref) <= (terms + 2) * EPS * bound)
