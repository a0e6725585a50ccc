"""The stored products at the edges of their tiling: row counts around a wave and
a workgroup, rows of no element, rows longer than the window in which a wave
stages its rows, rows of which only some fit it, and several vectors; explicit
and packed elements.

Rows are written by hand into the stored-matrix struct.  Tolerance of a row:
(n + 2) eps sum |a v| with n its element count."""
import ctypes

import numpy as np
import pytest

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


def _lengths(name, dim, rng):
    if name == "even":
        return rng.integers(20, 37, dim)
    if name == "sparse":
        return rng.integers(0, 3, dim)
    if name == "mixed":           # one row in 40 far longer than the others
        n = rng.integers(0, 12, dim)
        n[rng.integers(0, dim, max(1, dim // 40))] = 900
        return n
    n = np.zeros(dim, dtype=np.int64)   # all elements in one row, past the largest window
    n[dim // 2] = 5000
    return n


@pytest.mark.parametrize("name", ["even", "sparse", "mixed", "one"])
@pytest.mark.parametrize("dim", [1, 63, 64, 65, 257, 1000, 140001])
@pytest.mark.parametrize("packed", [False, True])
def test_rows(q, name, dim, packed):
    import torch
    from paper_2305_18643_amd import _binding as B
    print(f"rows {name} dim {dim} packed {packed}", flush=True)
    rng = np.random.default_rng(dim)
    n = np.asarray(_lengths(name, dim, rng), dtype=np.int64)
    rowptr = np.concatenate([[0], np.cumsum(n)])
    nnz = int(rowptr[-1])
    col = rng.integers(0, dim, nnz).astype(np.uint32)
    table = np.sort(rng.uniform(-2, 2, 64))
    idx = rng.integers(0, 64, nnz)
    val = table[idx]
    nvec = 2
    v = rng.uniform(-1, 1, (nvec, dim))
    dev = [torch.tensor(rowptr, device="cuda"), torch.tensor(col.view(np.int32), device="cuda"),
           torch.tensor(val, device="cuda"),
           torch.tensor((col | (idx.astype(np.uint32) << 26)).view(np.int32), device="cuda"),
           torch.tensor(table, device="cuda")]
    h = B.SymCsrC()
    h.dim, h.nnz = dim, nnz
    h.rowptr, h.col, h.val = (t.data_ptr() if t.numel() else None for t in dev[:3])
    if packed:
        if nnz == 0:
            pytest.skip("nothing to pack")
        h.packed, h.table = dev[3].data_ptr(), dev[4].data_ptr()
    buf = torch.full((nvec * dim + 256,), 7.5, dtype=torch.float64, device="cuda")
    w = buf[128:128 + nvec * dim]
    x = torch.tensor(v, device="cuda").reshape(-1)
    lib = q.load_library()
    rc = lib.qcm_sym_hv(ctypes.byref(h), ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(w.data_ptr()),
                        nvec, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    assert bool((buf[:128] == 7.5).all()) and bool((buf[128 + nvec * dim:] == 7.5).all())
    got = w.cpu().numpy().reshape(nvec, dim)
    row = np.repeat(np.arange(dim), n)
    for k in range(nvec):
        p = val.astype(np.longdouble) * v[k][col]
        ref = np.zeros(dim, dtype=np.longdouble)
        mag = np.zeros(dim)
        np.add.at(ref, row, p)
        np.add.at(mag, row, np.abs(p).astype(float))
        assert np.all(np.abs(got[k] - ref) <= (n + 2) * EPS * mag)
