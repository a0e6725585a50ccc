"""The hop lists of the down strings, stored row by row: one to more than 64
bonds, on both sides of each lane count a row is built with, and row counts that
leave groups of lanes idle; and the time to build them against the lists of the
up strings, which hold the same entries slot by slot.

The products are of small integers, which no order of the sums rounds: they are
exact.  The two list builders do the same work, so a plan of mirrored sectors may
cost at most twice as much either way."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    q.load_library()
    return q


def _model(nbond, L):
    """L orbitals with exactly nbond bonds."""
    rng = np.random.default_rng(950 + nbond)
    a, b = np.triu_indices(L, 1)
    on = np.sort(rng.permutation(a.size)[:nbond])
    t = np.diag(rng.integers(-9, 10, L).astype(float))
    t[a[on], b[on]] = t[b[on], a[on]] = rng.integers(1, 99, nbond)
    return t, rng.integers(0, 9, L).astype(float)


@pytest.mark.parametrize("nbond", [0, 1, 7, 8, 9, 16, 17, 32, 33, 64, 65, 66])
@pytest.mark.parametrize("nup,ndn", [(0, 1), (1, 5), (2, 6), (5, 5)])
def test_product(q, nbond, nup, ndn):
    import torch
    print(f"hop lists {nbond} bonds ({nup},{ndn})", flush=True)
    t, U = _model(nbond, 12)
    m = (t, U)
    b = q.sector_basis(12, nup, ndn)
    x = np.random.default_rng(5).integers(-999, 1000, b.dim).astype(float)
    v = torch.tensor(x, device="cuda")
    w = torch.full_like(v, 7.5)
    q.HvPlan(m, b, "fp64")(v, w)
    assert np.array_equal(w.cpu().numpy(), oracle.hv(t, U, nup, ndn, x))


def test_time_of_a_plan(q):
    import torch
    t, U = _model(190, 20)
    m = (t, U)

    def plan(nup, ndn):
        b = q.sector_basis(20, nup, ndn)
        ts = []
        for k in range(24):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            q.HvPlan(m, b, "fp64").close()
            torch.cuda.synchronize()
            if k > 3:
                ts.append(time.perf_counter() - t0)
        return min(ts)

    rows, slots = plan(1, 10), plan(10, 1)
    print(f"plan: row by row {rows * 1e6:.0f} us, slot by slot {slots * 1e6:.0f} us", flush=True)
    assert rows < 2 * slots


@pytest.mark.parametrize("nbond", [0, 3, 17, 66])
@pytest.mark.parametrize("nup,ndn", [(0, 0), (0, 6), (12, 5), (12, 12)])
@pytest.mark.parametrize("nvec", [1, 7])
def test_one_up_string(q, nbond, nup, ndn, nvec):
    """A single up string: the lists of the down strings slot by slot."""
    import torch
    t, U = _model(nbond, 12)
    b = q.sector_basis(12, nup, ndn)
    x = np.random.default_rng(6).integers(-999, 1000, (nvec, b.dim)).astype(float)
    v = torch.tensor(x.reshape(-1), device="cuda")
    w = torch.full_like(v, 7.5)
    q.HvPlan((t, U), b, "fp64")(v, w, nvec)
    got = w.cpu().numpy().reshape(nvec, b.dim)
    for k in range(nvec):
        assert np.array_equal(got[k], oracle.hv(t, U, nup, ndn, x[k]))


def test_time_of_one_up_string(q):
    """2,704,156 rows of one string.  The lists are read once, at the rate of a
    copy; the gathers take as long again, and half of both is allowed on top."""
    import torch
    L = 24
    t = np.zeros((L, L))
    for k in range(L):
        t[k, (k + 1) % L] = t[(k + 1) % L, k] = -1.0
    b = q.sector_basis(L, 0, 12)
    v = torch.rand(b.dim, device="cuda", dtype=torch.float64)
    w = torch.empty_like(v)
    plan = q.HvPlan((t, np.full(L, 4.0)), b, "fp64")
    hops = 12 * 2 * L * oracle.binom(L - 2, 11)      # bytes
    src = torch.zeros(hops // 2, dtype=torch.uint8, device="cuda")      # read and written
    dst = torch.empty_like(src)

    def best(f):
        ts = []
        for k in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                f()
            torch.cuda.synchronize()
            ts.append((time.perf_counter() - t0) / 10)
        return min(ts)

    product, copy = best(lambda: plan(v, w)), best(lambda: dst.copy_(src))
    print(f"product {product * 1e6:.0f} us, copy {copy * 1e6:.0f} us", flush=True)
    assert product < 3 * copy
