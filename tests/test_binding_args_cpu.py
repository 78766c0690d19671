"""Argument forms the binding packs itself: operator parameters from any
iterable, and term lists, against descriptors filled field by field."""
import ctypes

import numpy as np
import pytest

import paper_1207_1746_amd as G


@pytest.mark.parametrize("make", [tuple, list, np.array, iter, lambda v: np.array(v, dtype=np.float32),
                                  lambda v: (x for x in v)])
@pytest.mark.parametrize("p", [(), (0.0,), (0.5,), (0.75, 0.0, 4), (1, 2, 3, 4, 5, 6, 7, 8)])
def test_parameters_from_any_iterable(make, p):
    sd = G._stencil(G.K_WJACOBI_TB, make(p))
    assert sd.kind == G.K_WJACOBI_TB
    assert list(sd.p) == list(p) + [0.0] * (8 - len(p))


def test_parameters_from_a_tensor():
    torch = pytest.importorskip("torch")
    assert list(G._stencil(G.K_WJACOBI, torch.tensor([0.5, 0.25])).p)[:2] == [0.5, 0.25]


def test_parameters_refused():
    with pytest.raises(TypeError):
        G._stencil(G.K_WJACOBI, None)
    with pytest.raises(IndexError):
        G._stencil(G.K_WJACOBI, range(9))


@pytest.mark.parametrize("terms", [
    [], [(0, 1, -1, 2, 3, 0.5, -1)], [(0, 0, 0, 0, 0, 1, -1), (1, 2, -2 ** 31, 2 ** 31 - 1, 4, -0.0, 3)],
    [(np.int64(0), np.int32(1), 1, 0, 0, np.float32(0.1), -1)], [(0, 0, 2 ** 32 + 1, 0, 0, "0.5", -1)],
])
def test_terms_match_fields(terms):
    arr = G._terms(terms)
    assert len(arr) == len(terms)
    for a, (o, g, dx, dy, dz, w, coef) in zip(arr, terms):
        want = G.Term()
        want.out, want.grid, want.dx, want.dy, want.dz, want.coef = o, g, dx, dy, dz, coef
        want.w = float(w)
        assert bytes(a) == bytes(want)
    with pytest.raises(TypeError):
        G._terms([(0, 0, 0.5, 0, 0, 1.0, -1)])
