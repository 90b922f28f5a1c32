"""Modes >= 2 whose lanes load and store neighbouring columns together, with
every tile that does so (SETD_TILE_MODEB forces one), on matrices read as they
are given: columns in whole groups and not, slabs that end between tiles and
inside them, fewer columns than a group holds, contractions of one and two
chunks of 8 with every kind of remainder, tensors that are only 8-byte aligned,
a base, NaN in one fibre; and the shapes whose tile the launcher chooses by
other rules (one block of i, a full chip, a matrix past the L2).

Tolerance: the products' 1e-13 of the largest entry (n <= 300 products of
uniform entries, each rounded to 2^-53); 1e-12 for n up to 2100."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

TOL = 1e-13
TILES = ["1x4x1", "2x2x1", "4x2x1", "5x2x1", "4x4x1"]
# (dims, mode): na = product of the sizes before the mode, nb of those after it
SHAPES = [((4, 3, 5), 1), ((8, 8, 7), 1), ((6, 16, 9), 1), ((3, 5, 4), 1), ((64, 2, 9), 1), ((68, 9, 3), 1), ((12, 17, 6), 1),
          ((132, 31, 2), 1), ((9, 7, 2), 2), ((3, 1, 4), 2), ((5, 13, 16), 2), ((16, 16, 1), 2), ((50, 3, 33), 2),
          ((2, 1, 8), 2), ((260, 100, 2), 1)]


def _unaligned(x):
    t = torch().empty(x.size + 1, dtype=torch().float64, device="cuda")[1:]
    t.copy_(dev(x))
    return t


@pytest.mark.parametrize("tile", TILES)
def test_neighbouring_columns(tile, monkeypatch):
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for dims, mu in SHAPES:
        say("columns", tile, dims, "mode", mu + 1)
        T, W0, L = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2), wl.random_matrix(dims[mu], 3, scale=0.3)
        mats = [None] * 3
        mats[mu] = dev(L)
        V, W = _unaligned(T), _unaligned(W0)
        ref = oracle.mode_product(T, L, mu + 1)
        setd.tucker_apply(V, W, dims, mats, alpha=0.7, beta=1.0)
        assert rel_err(host(W, dims), 0.7 * ref + W0) < TOL, (dims, mu)
        W.fill_(float("nan"))
        setd.tucker_apply(V, W, dims, mats)
        assert rel_err(host(W, dims), ref) < TOL, (dims, mu)


@pytest.mark.parametrize("tile", TILES)
def test_nan_stays_in_its_column(tile, monkeypatch):
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for dims, mu, at in [((8, 13, 5), 1, (7, 12, 4)), ((8, 13, 5), 1, (0, 3, 2)), ((7, 9, 11), 2, (6, 8, 10)),
                         ((4, 8, 3), 1, (2, 0, 1))]:
        T = wl.random_tensor(dims, 9)
        T[at] = np.nan
        mats = [None] * 3
        mats[mu] = dev(wl.random_matrix(dims[mu], 4))
        W = torch().empty(T.size, dtype=torch().float64, device="cuda")
        setd.tucker_apply(dev(T), W, dims, mats)
        bad = np.zeros(dims, dtype=bool)
        line = list(at)
        line[mu] = slice(None)
        bad[tuple(line)] = True
        assert np.array_equal(np.isnan(host(W, dims)), bad), (tile, dims)


@pytest.mark.parametrize("dims,mu,tol", [
    ((1, 40, 70), 0, TOL), ((96, 2, 300), 1, TOL), ((96, 16, 40), 1, TOL), ((97, 17, 40), 1, TOL),   # one block of i, two
    ((64, 1030, 64), 0, TOL), ((60, 1030, 64), 0, TOL), ((128, 520, 128), 2, TOL),                    # a full chip
    ((641, 50), 0, 1e-12), ((40, 650), 1, 1e-12), ((2100, 700), 0, 1e-12), ((700, 2100), 1, 1e-12)])  # past the L2
def test_chosen_tile(dims, mu, tol):
    T, L = wl.random_tensor(dims, 5), wl.random_matrix(dims[mu], 6, scale=0.3)
    mats = [None] * len(dims)
    mats[mu] = dev(L)
    W = torch().empty(T.size, dtype=torch().float64, device="cuda")
    say("chosen tile", dims, "mode", mu + 1)
    setd.tucker_apply(dev(T), W, dims, mats)
    assert rel_err(host(W, dims), oracle.mode_product(T, L, mu + 1)) < tol
