"""Band Lanczos at the edges of the one-launch step for vectors of one chunk:
sectors of one state, of a few, of less and more than a chunk, one start state
and several, and parts that end early.

Against the oracle's recurrence from the same start states: the same R, Lambda
and G to 1e-8, Q Q^T = 1 to 1e-12 where both parts exist."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

Z = synth.omega_grid()


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    q.load_library()
    return q


CASES = [(synth.random_model(901, 2, 1, 0), [0]),              # electron part: one state
         (synth.random_model(902, 2, 1, 1), [0, 1]),
         (synth.random_model(903, 5, 2, 2), [1]),
         (synth.random_model(904, 5, 2, 2), [0, 1, 2, 3, 4]),
         (synth.random_model(906, 13, 4, 1), [0, 3, 6]),       # 16,731 and 3,718
         (synth.random_model(907, 7, 7, 3), [0, 1])]           # no electron part


@pytest.mark.parametrize("m,orbs", CASES, ids=lambda x: getattr(x, "name", None))
def test_band_steps(q, m, orbs):
    import torch
    from oracle import band
    print(f"band {m.name} ({m.nup},{m.ndn}) p={len(orbs)}", flush=True)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    ro = oracle.lanczos_gs(m.t, m.U, m.nup, m.ndn, want_vector=True)
    psi = torch.from_numpy(ro["psi"]).to("cuda")
    g = q.green_band(m, b, psi, ro["e0"], orbs, Z, max_basis=16)
    Go, parts = band.green_band(m.t, m.U, m.nup, m.ndn, ro["psi"], orbs, ro["e0"], Z, max_basis=16)
    for k in range(2):
        assert g["R"][k] == parts[k][0].shape[0]
        assert np.abs(np.sort(g["lam"][k]) - np.sort(parts[k][0])).max(initial=0.0) <= 1e-8
    assert np.abs(g["G"].cpu().numpy() - Go).max() <= 1e-8
    if 0 < m.nup < m.L:
        Q = np.concatenate(g["Q"], axis=1)
        assert np.abs(Q @ Q.T - np.eye(len(orbs))).max() <= 1e-12
