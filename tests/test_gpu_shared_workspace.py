"""A ground-state call whose start vector and result lie in the same buffer as
its workspace, past the bytes it needs: the result of separate buffers."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32v"])
@pytest.mark.parametrize("inside", ["psi", "v0", "both"])
def test_vectors_past_the_workspace(prec, inside):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_18643_amd as q
    from paper_2305_18643_amd import _binding as B
    lib = q.load_library()
    m = synth.chain(8, U=4.0, mu=2.0)
    b = q.sector_basis(m.L, m.nup, m.ndn)
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = torch.tensor(np.random.default_rng(51).uniform(-1, 1, b.dim), dtype=dt, device="cuda")
    want = q.lanczos_gs(m, b, prec=prec, fixed_steps=40, v0=x)
    hm = B.as_model(m)
    o = B.LanczosOpts()
    lib.qcm_lanczos_default_opts(ctypes.byref(o))
    o.fixed_steps, o.prec = 40, B.PREC[prec]
    need = ctypes.c_size_t(0)

    def call(d_gs, d_ws, n):
        res = B.GsResult()
        rc = lib.qcm_lanczos_gs(ctypes.byref(hm.c), ctypes.byref(b.c), ctypes.byref(o), None, None, d_gs,
                                ctypes.byref(res), d_ws, n, ctypes.byref(need), None)
        assert rc == 0, lib.qcm_last_error()
        return res
    call(None, None, 0)
    at = -(-need.value // 256) * 256
    buf = torch.zeros(at + 60 * 8 * b.dim, dtype=torch.uint8, device="cuda")
    psi = torch.zeros(b.dim, dtype=torch.float64, device="cuda")
    v0 = x
    if inside in ("psi", "both"):
        lo = at + 9 * 8 * b.dim + 512
        psi = buf[lo // 8 * 8:][:8 * b.dim].view(torch.float64)
    if inside in ("v0", "both"):
        lo = (at + 21 * 8 * b.dim) // 8 * 8
        v0 = buf[lo:][:x.element_size() * b.dim].view(dt)
        v0.copy_(x)
    o.d_v0 = v0.data_ptr()
    torch.cuda.synchronize()
    r = call(psi.data_ptr(), buf.data_ptr(), buf.numel())
    torch.cuda.synchronize()
    assert r.e0 == want["e0"] and r.n_iter == 40
    assert torch.equal(psi, want["psi"])
    assert torch.equal(v0, x)
