"""Recurrences longer than the tridiagonal test keeps in LDS (640 steps): fixed
steps around that length and tests after every step, every 50th and with none
before the last, against scipy's eigen-solver of the returned coefficients.

H without hopping on states of about evenly spread energies (the start vector
is zero on the others), so that the lowest Ritz value has not converged, no
orthogonality is lost and the residual of the Ritz vector is beta |s_last|.
Tolerances: Ritz values 1e-14 of |T| = 10 times a few; with the lowest pair 1e-5
apart an eigenvector carries 2 eps |T| / 1e-5 = 2e-10, so its last component times
beta, and the residual of psi, 1e-9."""
import numpy as np
import pytest
from scipy.linalg import eigh_tridiagonal

import oracle
import synth

pytestmark = pytest.mark.gpu

L, NUP, NDN = 12, 6, 5


@pytest.fixture(scope="module")
def problem():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    rng = np.random.default_rng(62)
    eps = np.sort(rng.uniform(0, 1, L))

    def energies(n):
        s = oracle.sector_states(L, n)
        return ((s[:, None] >> np.arange(L)) & 1) @ eps
    e = (energies(NDN)[:, None] + energies(NUP)[None, :]).ravel()
    v0 = rng.uniform(0.5, 1, e.size) * (np.abs(e - e.mean()) < 0.7 * e.std())
    m = synth.Model("levels", np.diag(eps), np.zeros(L), NUP, NDN)
    return q, m, q.sector_basis(L, NUP, NDN), torch.tensor(v0, device="cuda")


@pytest.mark.parametrize("kw", [dict(fixed_steps=n) for n in (639, 640, 641, 648, 1000)] +
                         [dict(max_iter=700, check_every=n, tol=-1.0) for n in (1, 50, 700)],
                         ids=lambda k: "_".join(f"{a}{b}" for a, b in k.items()))
def test_long_recurrence(problem, kw):
    q, m, b, v0 = problem
    print(f"long recurrence {kw}", flush=True)
    r = q.lanczos_gs(m, b, v0=v0, **kw)
    M = kw.get("fixed_steps", kw.get("max_iter"))
    assert r["n_iter"] == M and not r["breakdown"]
    th, s = eigh_tridiagonal(r["alpha"], r["beta"][:-1], select="i", select_range=(0, 1))
    assert th[1] - th[0] > 1e-5
    assert abs(r["e0"] - th[0]) <= 1e-13 and abs(r["theta1"] - th[1]) <= 1e-13
    est = r["beta"][-1] * abs(s[-1, 0])
    assert est > 1e-8
    assert abs(r["residual_est"] - est) <= 1e-9
    assert abs(r["true_residual"] - est) <= 1e-9
    assert abs(float(r["psi"].norm()) - 1.0) <= 1e-12


def test_a_test_that_ends_it_past_640_steps(problem):
    """Stopped by the residual at a tolerance met between 640 and 1000 steps."""
    q, m, b, v0 = problem
    for every in (1, 7):
        r = q.lanczos_gs(m, b, v0=v0, max_iter=1200, tol=1e-7, check_every=every)
        M = r["n_iter"]
        assert r["converged"] and 641 < M < 1100 and M % every == 0
        th, s = eigh_tridiagonal(r["alpha"], r["beta"][:-1], select="i", select_range=(0, 0))
        est = r["beta"][-1] * abs(s[-1, 0])
        assert est <= 1e-7 * max(1.0, abs(th[0])) + 1e-9
        assert abs(r["residual_est"] - est) <= 1e-9 and abs(r["true_residual"] - est) <= 1e-9
