"""The ground-state call with room for all, some or none of the recurrence's
vectors: the same bits whether the ground state is summed from kept vectors,
from kept ones and a rerun of the rest, or from a second pass; with residual
tests every step or every third, stopped by the test, by the step limit, by a
breakdown, or after fixed steps."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    q.load_library()
    return q


CASES = [(synth.chain(8, U=4.0, mu=2.0), dict()),
         (synth.chain(8, U=4.0, mu=2.0), dict(check_every=3)),
         (synth.chain(9, U=4.0, mu=2.0, nup=5, ndn=4), dict(prec="fp32v", reorth=1, tol=1e-7)),
         (synth.random_model(801, 9, 4, 4), dict(max_iter=17)),
         (synth.random_model(801, 9, 4, 4), dict(fixed_steps=21)),
         (synth.rect_cluster(4, 4, U=8.0, mu=4.0, nup=8, ndn=1), dict()),   # two-pass product
         (synth.rect_cluster(4, 4, U=8.0, mu=4.0, nup=8, ndn=1), dict(prec="fp32v", reorth=1, fixed_steps=15)),
         (synth.two_site(U=4.0), dict()),                                   # breakdown after 3 steps
         (synth.rect_cluster(3, 1, t=0.0, U=5.0, mu=1.0, nup=2, ndn=1), dict())]


@pytest.mark.parametrize("m,kw", CASES, ids=[f"{m.name}_{m.nup}_{m.ndn}_{'_'.join(map(str, kw.values()))}" for m, kw in CASES])
def test_same_bits(q, m, kw, monkeypatch):
    from paper_2305_18643_amd import _binding as B
    print(f"kept vectors {m.name} ({m.nup},{m.ndn}) {kw}", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    got = []
    for keep in (0, 5, 160):
        monkeypatch.setattr(B, "_KEEP_VECTORS", keep)
        got.append(q.lanczos_gs(m, b, **kw))
    for r in got[1:]:
        for k in ("e0", "residual_est", "true_residual", "n_iter", "converged", "breakdown"):
            assert r[k] == got[0][k], (k, r[k], got[0][k])
        for k in ("alpha", "beta"):
            assert np.array_equal(r[k], got[0][k])
        assert np.array_equal(r["psi"].cpu().numpy(), got[0]["psi"].cpu().numpy())


@pytest.mark.parametrize("m", [synth.chain(8, U=4.0, mu=2.0), synth.random_model(801, 9, 4, 4)], ids=["chain8", "rand9"])
def test_step_count_of_the_oracle(q, m):
    """Steps enqueued past the one that met the test leave no trace."""
    b = q.sector_basis(m.L, m.nup, m.ndn)
    r = q.lanczos_gs(m, b)
    o = oracle.lanczos_gs(m.t, m.U, m.nup, m.ndn)
    assert abs(r["n_iter"] - o["n_iter"]) <= 1 and r["converged"]
    assert abs(r["e0"] - o["e0"]) <= 1e-10 * abs(o["e0"])
    assert r["alpha"].shape == (r["n_iter"],)
