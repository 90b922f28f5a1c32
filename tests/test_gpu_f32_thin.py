"""FP32 products along modes of up to 16 and a little more (one block of i, whose
lanes hold four columns): the same bits as with 1 x 1 tiles, which hold one; the
columns in whole groups of four and not, several slabs, fewer columns than a
group, a NaN in one fibre.  Against the oracle 1e-5 of the largest entry (2^-24
times sums of up to 17 terms, and the rounding of the input)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

SHAPES = [((4, 3, 5), 1), ((8, 16, 7), 1), ((6, 16, 9), 1), ((3, 5, 4), 1), ((64, 2, 9), 1), ((68, 9, 3), 1), ((132, 1, 70), 1),
          ((9, 7, 2), 2), ((3, 1, 4), 2), ((5, 13, 16), 2), ((50, 3, 12), 2), ((2, 1, 8), 2), ((1, 3, 6), 2), ((36, 17, 5), 1)]


@pytest.mark.parametrize("dims,mu", SHAPES)
def test_same_bits(dims, mu, monkeypatch):
    T, W0, L = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2), wl.random_matrix(dims[mu], 3, scale=0.3)
    mats = [None] * 3
    mats[mu] = dev(L)
    ref = 0.7 * oracle.mode_product(T, L, mu + 1) + W0
    got = {}
    for tile in ("1x1", "1x4", None):
        if tile is None:
            monkeypatch.delenv("SETD_TILE_F32_MODEB")
        else:
            monkeypatch.setenv("SETD_TILE_F32_MODEB", tile)
        W = dev(W0)
        setd.tucker_apply(dev(T), W, dims, mats, alpha=0.7, beta=1.0, prec=setd.PREC_F32)
        got[tile] = host(W, dims)
        say("f32 thin", dims, mu, tile, "rel_inf %.2e" % rel_err(got[tile], ref))
        assert rel_err(got[tile], ref) < 1e-5
        assert np.array_equal(got[tile], got["1x1"])
        X = T.copy()
        at = tuple(n - 1 for n in dims)
        X[at] = np.nan
        setd.tucker_apply(dev(X), W, dims, mats, prec=setd.PREC_F32)
        bad = np.zeros(dims, dtype=bool)
        bad[tuple(slice(None) if k == mu else at[k] for k in range(3))] = True
        assert np.array_equal(np.isnan(host(W, dims)), bad)
