"""The k sum of the pole formula at the edges of its kernel: one to 64 poles,
one to eight sites, already diagonal L(k), all poles of one sign, against
numpy's eigvalsh of the same L(k).  Both are backward stable: the sum of at most
R eigenvalues is held to 8 R eps |L(k)|_F."""
import numpy as np
import pytest

from oracle import vca as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,R,kind", [(1, 1, "rand"), (2, 2, "rand"), (4, 3, "rand"), (8, 24, "rand"), (4, 31, "rand"),
                                      (3, 33, "rand"), (8, 63, "rand"), (8, 64, "rand"), (4, 12, "diagonal"),
                                      (4, 16, "positive"), (4, 64, "negative")])
def test_per_k_sums(L, R, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    rng = np.random.default_rng(100 * L + R)
    poles = np.sort(rng.uniform(-8, 8, R))
    if kind == "positive":
        poles = 40 + np.abs(poles)
    if kind == "negative":
        poles = -40 - np.abs(poles)
    Q = np.zeros((L, R)) if kind == "diagonal" else rng.normal(size=(L, R)) / np.sqrt(R)
    dt = rng.normal(size=(L, L))
    dt = 0.5 * (dt + dt.T)
    bonds = [(int(rng.integers(L)), int(rng.integers(L)), (int(rng.integers(-2, 3)), 1, 0), float(rng.normal()))
             for _ in range(5)]
    ks = rng.uniform(0, 1, (7, 3))
    om, per = q.vca_omega(0.5, poles, Q, dt, bonds, ks)
    ref = np.zeros(7)
    for i, k in enumerate(ks):
        Lk = np.diag(poles) + Q.T @ O.v_of_k(L, dt, bonds, k) @ Q
        w = np.linalg.eigvalsh(0.5 * (Lk + Lk.conj().T))
        ref[i] = w[w < 0].sum()
        assert abs(per[i] - ref[i]) <= 8 * R * 2.0 ** -53 * max(np.linalg.norm(Lk), 1.0), (per[i], ref[i])
    want = 0.5 + 2 * (ref.mean() - poles[poles < 0].sum())
    assert abs(om - want) <= 1e-12 * max(1.0, abs(want), np.abs(poles).sum())
