"""The workspace a ground-state call offers (host logic): room for the
recurrence's vectors, but only a small part of the card's free memory, and
none where that would hold only a few of them."""
from types import SimpleNamespace

import pytest

from paper_2305_18643_amd import _binding as B

NEED = 12345


class OutOfMemory(Exception):
    pass


def _torch(free, limit=None, held=0):
    """A stand-in whose empty() hands back the number of bytes asked for; held:
    bytes in its allocator that no tensor uses."""
    looked = []

    def empty(n, dtype=None, device=None):
        if limit is not None and n > limit:
            raise OutOfMemory
        return n

    def info(device=None):
        looked.append(device)
        return free, 288 << 30

    def stats(device=None):
        return {"reserved_bytes": {"all": {"current": (5 << 30) + held}}, "allocated_bytes": {"all": {"current": 5 << 30}}}
    return SimpleNamespace(empty=empty, uint8=None, OutOfMemoryError=OutOfMemory,
                           cuda=SimpleNamespace(mem_get_info=info, memory_stats_as_nested_dict=stats), looked=looked)


def _o(prec=B.QCM_FP64, want=1, max_iter=600, fixed=0):
    return SimpleNamespace(prec=prec, want_vector=want, max_iter=max_iter, fixed_steps=fixed)


def _kept(t, o, dim):
    vec = -(-dim * (8 if o.prec == B.QCM_FP64 else 4) // 256) * 256
    extra = B._gs_workspace(t, NEED, o, dim, "cuda:0") - NEED
    return (extra - 256) // vec if extra else 0


@pytest.mark.parametrize("dim,o,want", [(36, _o(), 160), (36, _o(max_iter=20), 21), (36, _o(fixed=9), 10), (36, _o(fixed=2), 0),
                                        (36, _o(want=0), 0), (853776, _o(), 160), (853776, _o(B.QCM_FP32V), 160),
                                        (11778624, _o(), 50), (11778624, _o(B.QCM_FP32V), 100), (165636900, _o(), 0),
                                        (41409225, _o(), 0)])
def test_vectors_kept_on_an_empty_card(dim, o, want):
    assert _kept(_torch(283 << 30), o, dim) == want


@pytest.mark.parametrize("free", [0, 1 << 30, 10 << 30, 100 << 30, 283 << 30])
@pytest.mark.parametrize("dim", [36, 63504, 853776, 11778624, 165636900])
@pytest.mark.parametrize("prec", [B.QCM_FP64, B.QCM_FP32V])
def test_a_small_part_of_the_free_memory(free, dim, prec):
    t = _torch(free)
    extra = B._gs_workspace(t, NEED, _o(prec), dim, "cuda:0") - NEED
    assert extra <= max(free // 64, 64 << 20) + 512
    assert t.looked == [] or t.looked == ["cuda:0"]


def test_memory_held_by_the_allocator_is_free():
    assert _kept(_torch(0, held=283 << 30), _o(), 11778624) == _kept(_torch(283 << 30), _o(), 11778624) == 50
    assert _kept(_torch(83 << 30, held=200 << 30), _o(), 11778624) == 50


def test_small_offers_do_not_look():
    t = _torch(0)
    assert _kept(t, _o(), 4900) == 160 and t.looked == []


def test_bare_workspace_when_the_offer_does_not_fit():
    assert B._gs_workspace(_torch(283 << 30, limit=1 << 20), NEED, _o(), 853776, "cuda:0") == NEED
