"""Ground-state calls whose recurrence ends before its last allowed step: a
fixed number of steps from a vector in a small invariant subspace, and residual
tests several steps apart."""
import time

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


@pytest.mark.parametrize("L,nup,ndn", [(6, 3, 3), (14, 7, 7), (16, 8, 1)])   # fused, long rows, two-pass
@pytest.mark.parametrize("steps", [1, 2, 3, 200])
def test_fixed_steps_from_an_eigenvector(q, L, nup, ndn, steps):
    """H without hopping: any basis state is an eigenvector, so the chain stops
    after its first step whatever the number asked for."""
    import torch
    m = synth.chain(L, t=0.0, U=4.0, mu=1.0)
    b = q.sector_basis(L, nup, ndn)
    v0 = torch.zeros(b.dim, dtype=torch.float64, device="cuda")
    v0[b.dim // 3] = 1.0
    r = q.lanczos_gs(m, b, fixed_steps=steps, v0=v0)
    e = oracle.hv_rows(m.t, m.U, nup, ndn, v0.cpu().numpy(), np.array([b.dim // 3]))[0]
    assert r["n_iter"] == 1 and r["breakdown"] and r["converged"]
    assert r["alpha"].shape == (1,) and abs(r["e0"] - e) <= 1e-12 * max(1.0, abs(e))
    assert torch.equal(r["psi"].abs(), v0)


@pytest.mark.parametrize("m,want", [(synth.two_site(U=4.0), None), (synth.random_model(921, 6, 1, 0), 6)],
                         ids=["two_site", "one_electron"])
@pytest.mark.parametrize("check_every", [1, 7])
def test_fixed_steps_small_krylov_space(q, m, want, check_every):
    """More steps than the sector has states: stopped at the same length as the
    chain that may stop by itself, with the same coefficients."""
    b = q.sector_basis(m.L, m.nup, m.ndn)
    r = q.lanczos_gs(m, b, fixed_steps=90, check_every=check_every)
    s = q.lanczos_gs(m, b, max_iter=90, tol=0.0)
    assert r["breakdown"] and r["n_iter"] == s["n_iter"] <= b.dim + 1
    if want:
        assert abs(r["n_iter"] - want) <= 1
    assert np.array_equal(r["alpha"], s["alpha"]) and np.array_equal(r["beta"], s["beta"])
    assert r["e0"] == s["e0"]


def test_time_of_a_chain_that_stops_at_once(q):
    """64 fixed steps cost no more than a few where the chain stops at the first
    (carried on to the end they cost five times as much as these four)."""
    import torch
    m = synth.chain(14, t=0.0, U=4.0, mu=1.0)
    b = q.sector_basis(14, 7, 7)
    v0 = torch.zeros(b.dim, dtype=torch.float64, device="cuda")
    v0[12345] = 1.0
    best = {}
    for steps in (4, 64):
        def call():
            q.lanczos_gs(m, b, fixed_steps=steps, want_vector=False, v0=v0)
        call()
        ts = []
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call()
            ts.append(time.perf_counter() - t0)
        best[steps] = min(ts)
    print(f"stops at once: {best[4] * 1e3:.2f} ms for 4 steps, {best[64] * 1e3:.2f} ms for 64", flush=True)
    assert best[64] <= 2.0 * best[4]


@pytest.mark.parametrize("L,nup,ndn,ahead", [(8, 4, 4, 4), (14, 7, 7, 2)])
@pytest.mark.parametrize("check_every", [2, 7, 20])
def test_steps_past_the_test_that_ends_it(q, L, nup, ndn, ahead, check_every):
    """The workspace holds the coefficients of every step that was enqueued: at
    most a few lie past the last one that counts.  The result is that of a test
    after every step, taken on to the next test."""
    import torch
    m = synth.chain(L, U=4.0, mu=2.0)
    b = q.sector_basis(L, nup, ndn)
    one = q.lanczos_gs(m, b, want_vector=False)
    ws = torch.zeros((8 << 20) + 32 * b.dim, dtype=torch.uint8, device="cuda")
    r = q.lanczos_gs(m, b, want_vector=False, check_every=check_every, ws=ws)
    M = r["n_iter"]
    assert r["converged"] and not r["breakdown"]
    assert M == -(-one["n_iter"] // check_every) * check_every
    assert np.array_equal(r["alpha"][:one["n_iter"]], one["alpha"])
    x = ws[:ws.numel() // 8 * 8].view(torch.float64)
    a = torch.from_numpy(r["alpha"]).cuda()
    at = [int(i) for i in torch.nonzero(x == a[0]).ravel().cpu() if torch.equal(x[i:i + M], a)]
    assert len(at) == 1
    past = int((x[at[0] + M:at[0] + 600] != 0).long().cumprod(0).sum())
    print(f"{L} orbitals, a test every {check_every} steps: {past} steps past step {M}", flush=True)
    assert past <= ahead


@pytest.mark.parametrize("m", [synth.chain(8, U=4.0, mu=2.0), synth.two_site(U=4.0), synth.random_model(922, 9, 4, 4)],
                         ids=["chain8", "two_site", "rand9"])
@pytest.mark.parametrize("kw", [dict(max_iter=5, check_every=2), dict(max_iter=600, check_every=3),
                                dict(max_iter=33, check_every=50), dict(max_iter=40, check_every=40, tol=0.0)],
                         ids=lambda k: "_".join(map(str, k.values())))
def test_tests_apart_against_the_oracle(q, m, kw):
    """Stopped by the limit, by a test, by a breakdown between two tests."""
    b = q.sector_basis(m.L, m.nup, m.ndn)
    r = q.lanczos_gs(m, b, **kw)
    M = r["n_iter"]
    T = np.diag(r["alpha"]) + np.diag(r["beta"][:M - 1], 1) + np.diag(r["beta"][:M - 1], -1)
    th, sv = np.linalg.eigh(T)
    scale = np.abs(th).max()
    assert abs(r["e0"] - th[0]) <= 1e-13 * scale
    if M > 1:
        assert abs(r["theta1"] - th[1]) <= 1e-13 * scale
    assert abs(r["residual_est"] - r["beta"][M - 1] * abs(sv[-1, 0])) <= 1e-12 * scale
    assert M == kw["max_iter"] or r["breakdown"] or M % kw["check_every"] == 0
    if r["converged"]:
        o = oracle.lanczos_gs(m.t, m.U, m.nup, m.ndn)
        assert abs(r["e0"] - o["e0"]) <= 1e-10 * max(1.0, abs(o["e0"]))


CHILD = """
import ctypes, sys, time
hip = ctypes.CDLL("libamdhip64.so")
assert hip.hipSetDeviceFlags(ctypes.c_uint(4)) == 0      # hipDeviceScheduleBlockingSync
import torch
import paper_2305_18643_amd as q, synth
m = synth.rect_cluster(4, 4, U=8.0, mu=4.0)
b = q.sector_basis(16, 8, 7)
kw = dict(max_iter=12, tol=0.0, want_vector=False, check_every=int(sys.argv[1]))
q.lanczos_gs(m, b, **kw)
w, c = time.perf_counter(), time.thread_time()
for _ in range(3):
    q.lanczos_gs(m, b, **kw)
print("share", (time.thread_time() - c) / (time.perf_counter() - w))
"""


@pytest.mark.parametrize("check_every", [1, 4])
def test_waits_block_where_the_program_asks(q, check_every):
    """A program that has asked the runtime for blocking waits gets them: with
    steps of 3 ms the calling thread sleeps for most of the call (polling the
    events took all of it)."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(check_every)], capture_output=True, text=True, timeout=100,
                       cwd=root, env=dict(os.environ, PYTHONPATH=root))
    assert r.returncode == 0, r.stderr
    share = float(r.stdout.split("share")[1])
    print(f"tests every {check_every} steps: the thread ran for {share:.2f} of the call", flush=True)
    assert share < 0.5
