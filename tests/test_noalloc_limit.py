"""Which sectors the allocation-free product takes and refuses: the nearest on
both sides of its 32 MiB among random and chain models, with the table sizes of
the layout that set the limit.  A taken sector gets as far as the check for the
vectors; nothing is launched."""
import ctypes
from math import comb

import pytest

import synth
from paper_2305_18643_amd import _binding as B

LIMIT = 32 << 20
# L, model, nup, ndn, bytes of its tables
SECTORS = [(18, 0.5, 6, 5, LIMIT - 208768), (17, 0.5, 9, 5, LIMIT - 468208),
           (27, 1.0, 3, 24, LIMIT - 583476), (23, None, 19, 18, LIMIT - 993852),
           (16, 0.5, 7, 10, LIMIT - 1015776), (17, 1.0, 11, 17, LIMIT + 313092),
           (22, 1.0, 4, 0, LIMIT + 444420), (16, 0.5, 8, 6, LIMIT + 797472),
           (17, 0.5, 10, 11, LIMIT + 968992), (15, 1.0, 7, 7, 38310028)]


@pytest.mark.parametrize("L,density,nup,ndn,size", SECTORS)
def test_taken_or_refused(L, density, nup, ndn, size):
    lib = B.load_library()
    m = synth.chain(L, U=4.0, mu=2.0, nup=nup, ndn=ndn) if density is None else \
        synth.random_model(L * 7, L, nup, ndn, density=density)
    h = B.as_model(m)
    b = B.Basis()
    b.L, b.n_up, b.n_dn, b.d_up, b.d_dn = L, nup, ndn, comb(L, nup), comb(L, ndn)
    b.dim = b.d_up * b.d_dn
    for f, t in B.Basis._fields_:
        if t is ctypes.c_void_p:
            setattr(b, f, 4096)   # any non-NULL table: not read before the refusal
    rc = lib.qcm_hv_noalloc(ctypes.byref(h.c), ctypes.byref(b), 0, None, None, None)
    assert rc == (B.QCM_EWORKSPACE if size > LIMIT else B.QCM_EARG)
    want = b"static scratch" if size > LIMIT else b"NULL vector"
    assert want in lib.qcm_last_error()
