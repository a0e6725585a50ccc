"""Continued-fraction chains of small sectors, whose steps run in one launch,
against the batched engine, whose steps are separate launches with the same
order of every sum: coefficients, lengths and G are the same bits.

Sectors with one up string, one down string, two strings, one to sixty-four
product blocks and just past them, sizes on both sides of the LDS limit, chains
that end early, odd row lengths and hop counts off the unrolled group."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

Z = synth.omega_grid()[:8]


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    q.load_library()
    return q


MODELS = [synth.random_model(801, 6, 5, 3),                  # electron part: d_up = 1
          synth.random_model(802, 6, 1, 3),                  # hole part: d_up = 1
          synth.random_model(803, 7, 3, 0),                  # one down string
          synth.random_model(804, 3, 1, 1),                  # 9 states, chains end early
          synth.random_model(805, 4, 2, 2, uniform_U=True),
          synth.random_model(806, 8, 4, 4, density=1.0),     # 28 bonds
          synth.random_model(807, 9, 1, 4, uniform_U=True),  # 36 x 126: past LDS in FP64
          synth.random_model(808, 9, 3, 4, density=0.3),     # 36 x 126 and 126 x 126
          synth.random_model(809, 13, 1, 6),                 # hole: 1 x 1716; electron past a chunk
          synth.random_model(810, 13, 12, 1),                # 1 x 13 and 78 x 13
          synth.random_model(811, 12, 2, 1),                 # 220 x 12, 12 x 12
          synth.random_model(812, 16, 2, 1, density=0.4),    # 560 x 16: past a chunk
          synth.chain(10, U=4.0, mu=2.0, nup=2, ndn=1)]      # 120 x 10, one t


@pytest.mark.parametrize("m", MODELS, ids=lambda m: f"{m.name}_{m.nup}_{m.ndn}")
@pytest.mark.parametrize("prec,reorth", [("fp64", 0), ("fp64", 1), ("fp32v", 0), ("fp32v", 1)])
def test_one_launch_equals_separate_launches(q, m, prec, reorth):
    import torch
    steps = 40
    orbs = [0, 1, 2]
    print(f"chains {m.name} ({m.nup},{m.ndn}) {prec} reorth {reorth}", flush=True)
    tol = 1e-12 if prec == "fp64" else 1e-7
    psi = torch.zeros(oracle.binom(m.L, m.nup) * oracle.binom(m.L, m.ndn), dtype=torch.float64,
                      device="cuda")
    eng = q.Engine(1 << 28, prec=prec, reorth=reorth, gf_steps=steps, max_jobs=2, z=Z, tol=tol)
    assert eng.submit(q.JobSpec((m.t, m.U), m.nup, m.ndn, orbs=orbs, seed=1, tag=0, psi=psi))
    out = []
    while eng.step(16):
        out += list(eng.poll())
    out += list(eng.poll())
    eng.close()
    e = out[0]
    b = q.sector_basis(m.L, m.nup, m.ndn)
    g = q.green_cf((m.t, m.U), b, e["psi"], e["e0"], orbs, Z, max_steps=steps, prec=prec,
                   reorth=reorth)
    assert np.array_equal(e["len"], g["len"])
    assert np.array_equal(e["coef"], g["coef"])
    assert np.array_equal(e["G"], g["G"].cpu().numpy())
