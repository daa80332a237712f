"""The deposit at the edges of its tiles: sort tiles of 2048 particles, row tiles
that do not divide ny, single rows, the wrapped row and plane, runs longer than
the 256 positions a block walks at a time (first, between and last in a row),
one to three sort passes, more than 32 sort tiles.  Against the FP64 oracle.

Tolerance: a cell sums the same products as the oracle, in another order.  With
uniform particles that is a few tens of terms; in a cluster of m particles the
pieces of eight keep the error of the sum below (m / 8 + 8) units of 2^-53 of
the sum of magnitudes, the oracle's own serial sum below m units.  m <= 3000 and
q in [0.5, 1.5] (no cancellation): 3400 * 1.2e-16 = 4e-13 < 1e-12 of the largest
magnitude.
"""
import math

import numpy as np
import pytest

import oracle
from gpu_helpers import announce, dev, host
from paper_1601_05448_amd import poisson as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.load()
    yield


CASES = [
    ((4, 4, 4), 1), ((4, 4, 4), 2048), ((4, 4, 1024), 2049), ((4, 6, 1024), 4095), ((8, 1024, 4), 2047),
    ((64, 48, 96), 70000), ((32, 12, 768), 5000), ((256, 6, 512), 100000), ((128, 128, 128), 1),
]


@pytest.mark.parametrize("cluster", [0, 255, 257, 3000])
@pytest.mark.parametrize("shape,np_", CASES, ids=lambda c: str(c).replace(" ", ""))
def test_deposit_tiles(shape, np_, cluster):
    announce("deposit tiles", shape, np_, cluster)
    rng = np.random.default_rng(np_ + cluster)
    L = (5.0, 3.0, 2.0 * math.pi)
    h = (L[0] / shape[2], L[1] / shape[1], L[2] / shape[0])
    pos = [rng.uniform(-1.0, 2.0, (np_, 3)) * np.array(L)]
    # the first cell, the last one (its footprint wraps in every direction), one inside a row
    for i, j, k in ((0, 0, 0), (shape[2] - 1, shape[1] - 1, shape[0] - 1), (2, 1, 3)):
        pos.append((np.array([i, j, k]) + rng.uniform(0.5, 1.5, (cluster, 3))) * h)
    pos = np.concatenate(pos)
    pos = pos[rng.permutation(pos.shape[0])]
    q = rng.uniform(0.5, 1.5, pos.shape[0])
    want = oracle.deposit(shape, pos, q, L)
    hd = P.poisson_create(shape, L)
    try:
        outs = []
        for _ in range(2):
            out = dev(np.full(shape, np.nan))
            P.poisson_deposit(hd, dev(pos), dev(q), out)
            outs.append(host(out))
    finally:
        P.poisson_destroy(hd)
    assert np.max(np.abs(outs[0] - want)) <= 1e-12 * np.max(np.abs(want))
    assert np.array_equal(outs[0], outs[1])


def test_deposit_leaves_the_output_on_a_bad_position():
    announce("deposit bad position: output untouched")
    shape, L = (8, 8, 16), (1.0, 1.0, 1.0)
    pos = np.random.default_rng(3).uniform(0.0, 1.0, (3000, 3))
    pos[2999, 2] = np.nan
    h = P.poisson_create(shape, L)
    try:
        out = dev(np.full(shape, 7.0))
        with pytest.raises(P.PoissonError) as e:
            P.poisson_deposit(h, dev(pos), None, out)
        assert e.value.code == P.POISSON_EDOMAIN
        assert np.all(host(out) == 7.0)
    finally:
        P.poisson_destroy(h)
