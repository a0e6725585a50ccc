"""Products and Lanczos steps of sectors whose rows are shorter than a wave's 64
lanes (one column of two rows a lane): one string to 45 a row and the next
longer row, odd rows, rows left over by the blocks, vectors in one workgroup
of one wave, lists of every length mod 4, vectors of more than 2 GB; and the
time of such a product against that of longer rows.

Tolerances as for the product's other shapes: (terms + 2) eps (|H||v|)_i and one
rounding to FP32; coefficients of the first steps 1e-12 |H|."""
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
    return [synth.random_model(901, 14, 0, 7),                       # one string, two blocks
            synth.random_model(902, 14, 14, 6, uniform_U=True),
            synth.random_model(903, 2, 1, 1),
            synth.random_model(904, 4, 2, 2, density=1.0),           # one vector, 18 pairs
            synth.random_model(905, 5, 1, 2, density=1.0, uniform_U=True),
            synth.chain(8, U=4.0, mu=2.0, nup=1, ndn=4),             # 280 pairs: four waves
            synth.random_model(906, 13, 1, 5, density=1.0),          # 78 bonds
            synth.chain(16, U=4.0, mu=2.0, nup=1, ndn=7),
            synth.random_model(907, 8, 2, 4),                        # 28 strings
            synth.random_model(908, 7, 3, 3, density=0.3),           # 35 strings, 35 rows
            synth.random_model(909, 10, 8, 5),                       # 45 strings
            synth.random_model(910, 11, 2, 4)]                       # 55 strings: tiles


IDS = lambda m: f"{m.name}_{m.nup}_{m.ndn}"


def _tol(m, x, ref, prec):
    terms = 2 * int(np.count_nonzero(np.triu(m.t, 1))) + 3
    tol = (terms + 2) * EPS * oracle.hv_abs_bound(m.t, m.U, m.nup, m.ndn, x) + 1e-300
    if prec == "fp32v":
        tol = tol + 2.0 ** -24 * np.abs(ref) * (1 + 2.0 ** -20)
    return tol


@pytest.mark.parametrize("m", _models(), ids=IDS)
@pytest.mark.parametrize("prec", ["fp64", "fp32v"])
@pytest.mark.parametrize("nvec", [1, 3, 300])
def test_product(q, m, prec, nvec):
    import torch
    print(f"short rows {m.name} ({m.nup},{m.ndn}) {prec} x{nvec}", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    dt = torch.float64 if prec == "fp64" else torch.float32
    v = torch.tensor(np.random.default_rng(21).uniform(-1, 1, (nvec, b.dim)), dtype=dt)
    plan = q.HvPlan(m, b, prec)
    buf = torch.full((nvec * b.dim + 256,), 7.5, dtype=dt, device="cuda")
    w = buf[128:128 + nvec * b.dim]
    plan(v.cuda().reshape(-1), w, nvec)
    assert bool((buf[:128] == 7.5).all()) and bool((buf[128 + nvec * b.dim:] == 7.5).all())
    got = w.double().cpu().numpy().reshape(nvec, b.dim)
    for k in sorted({0, nvec // 2, nvec - 1}):
        x = v[k].double().numpy()
        ref = oracle.hv(m.t, m.U, m.nup, m.ndn, x)
        assert np.all(np.abs(got[k] - ref) <= _tol(m, x, ref, prec))


@pytest.mark.parametrize("m", [m for m in _models() if oracle.binom(m.L, m.nup) * oracle.binom(m.L, m.ndn) > 30], ids=IDS)
@pytest.mark.parametrize("reorth", [0, 1])
def test_first_lanczos_steps(q, m, reorth):
    import torch
    print(f"short rows steps {m.name} ({m.nup},{m.ndn})", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    x = np.random.default_rng(22).uniform(-1, 1, b.dim)
    r = q.lanczos_gs(m, b, fixed_steps=4, want_vector=False, reorth=reorth, v0=torch.tensor(x, device="cuda"))
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


def test_product_over_2gb_sampled_rows(q):
    """27 strings a row, 2.8 GB: neighbours through 64-bit addresses."""
    import torch
    m = synth.random_model(911, 27, 1, 11, density=0.12)
    print("short rows 27 orbitals (1,11)", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    assert b.d_up == 27 and b.dim * 8 > 2 ** 31
    v = oracle.start_vector(8, b.dim)
    rows = np.unique(np.concatenate([np.random.default_rng(23).integers(0, b.dim, 2000), np.arange(64),
                                     np.arange(b.dim - 64, b.dim)]))
    w = q.hv(m, b, torch.from_numpy(v).cuda())
    got = w[torch.from_numpy(rows).cuda()].cpu().numpy()
    del w
    ref = oracle.hv_rows(m.t, m.U, m.nup, m.ndn, v, rows)
    bound = oracle.hv_abs_bound(m.t, m.U, m.nup, m.ndn, v, rows)
    terms = 2 * int(np.count_nonzero(np.triu(m.t, 1))) + 3
    assert np.all(np.abs(got - ref) <= (terms + 2) * EPS * bound)


@pytest.mark.parametrize("L,nup,ndn,nvec", [(4, 2, 2, 166666), (8, 1, 4, 10714), (16, 0, 8, 400)])
def test_time_against_longer_rows(q, L, nup, ndn, nvec):
    """At most 6 times the product of as many elements in rows of 252 strings:
    the first is one workgroup a vector, the others have as many elements in a
    workgroup (as tiles along the row: 22, 6.5 and more times)."""
    import torch

    def best(L, nup, ndn, nvec):
        m = synth.chain(L, U=4.0, mu=2.0)
        b = q.sector_basis(L, nup, ndn)
        v = torch.rand(nvec * b.dim, dtype=torch.float64, device="cuda")
        w = torch.empty_like(v)
        plan = q.HvPlan(m, b, "fp64")
        plan(v, w, nvec)
        ts = []
        for _ in range(7):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(5):
                plan(v, w, nvec)
            e[1].record()
            torch.cuda.synchronize()
            ts.append(e[0].elapsed_time(e[1]))
        return min(ts) / 5e-3 / (nvec * b.dim)
    short, long = best(L, nup, ndn, nvec), best(10, 5, 5, 94)
    print(f"short rows {L} ({nup},{ndn}) x{nvec}: {1e6 * short:.2f} us per million elements, long rows {1e6 * long:.2f}",
          flush=True)
    assert short <= 6.0 * long
