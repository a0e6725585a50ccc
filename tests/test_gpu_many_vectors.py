"""A product of more vectors than one launch of the kernel takes threads for."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,nup,ndn,nvec", [(8, 3, 0, (1 << 23) + 3), (2, 1, 1, (1 << 26) + 3)],
                         ids=["eight_waves_a_vector", "one_wave_a_vector"])
def test_vectors_past_one_launch(L, nup, ndn, nvec):
    """FP32 vectors, the same five in turn: every one has its own's product."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    m = synth.chain(L, U=4.0, mu=2.0)
    b = q.sector_basis(L, nup, ndn)
    print(f"{nvec} vectors of {b.dim} states", flush=True)
    x = torch.tensor(np.random.default_rng(31).uniform(-1, 1, (5, b.dim)), dtype=torch.float32)
    v = x.cuda().repeat(nvec // 5 + 1, 1)[:nvec].contiguous()
    w = torch.full_like(v, 7.5)
    q.HvPlan(m, b, "fp32v")(v.reshape(-1), w.reshape(-1), nvec)
    first = w[:5].clone()
    for k in range(5):
        ref = oracle.hv(m.t, m.U, nup, ndn, x[k].double().numpy())
        assert np.abs(first[k].double().cpu().numpy() - ref).max() <= 2.0 ** -23 * np.abs(ref).max() + 1e-12
    for k in range(5):
        assert bool((w[k::5] == first[k]).all())
