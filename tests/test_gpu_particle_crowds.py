"""Deposits whose particles crowd some tiles of the grid, or all of them: many runs
per tile (more than a block takes at a time), more than one tile per block (also
uneven), more positions than one group of counts holds.  Against the FP64 oracle,
with repeated bits; and the time of a crowded deposit beside a uniform one's.

Tolerance: at most m = 6000 positive terms fall on a cell; summed in pieces of eight
their error is below (m / 8 + 8) units of 2^-53 of the sum, the oracle's serial sum
below m units: 6800 * 1.2e-16 = 8.2e-13 < 1e-12 of the largest magnitude."""
import math
import time

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


# (nz, ny, nx), particles, cells (z, y, x) that hold them, from a corner that wraps
CASES = [
    ((16, 16, 16), 300000, (16, 16, 16)),     # 1172 blocks of positions: two groups
    ((4, 8, 1024), 100000, (4, 8, 1024)),     # one row per tile
    ((128, 64, 512), 60000, (1, 64, 512)),    # a sheet: thousands of runs in a tile
    ((128, 64, 512), 60000, (128, 2, 64)),
    ((128, 64, 512), 60000, (2, 2, 60)),
    ((64, 128, 512), 30000, (3, 9, 13)),
    ((512, 64, 64), 200000, (512, 1, 64)),    # two tiles per block
    ((1024, 32, 768), 50000, (1, 32, 768)),   # three tiles per block, two in the last
]


@pytest.mark.parametrize("shape,n,cells", CASES, ids=lambda c: str(c).replace(" ", ""))
def test_deposit_crowds(shape, n, cells):
    announce("deposit crowds", shape, n, cells)
    rng = np.random.default_rng(n + sum(cells))
    L = (5.0, 3.0, 2.0 * math.pi)
    h = np.array([L[d] / shape[2 - d] for d in range(3)])
    pos = (rng.uniform(0.0, 1.0, (n, 3)) * np.array(cells[::-1]) - 0.5) * h
    q = rng.uniform(0.5, 1.5, n)
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


def _times(shape, pos, n_calls=9):
    import torch

    h = P.poisson_create(shape, (1.0, 1.0, 1.0))
    out = torch.empty(shape, dtype=torch.float64, device="cuda")
    ts = []
    try:
        for _ in range(n_calls):
            torch.cuda.synchronize()
            t = time.perf_counter()
            P.poisson_deposit(h, pos, None, out)
            ts.append(time.perf_counter() - t)
    finally:
        P.poisson_destroy(h)
    return sorted(ts)[len(ts) // 2]


@pytest.mark.parametrize("box", [(1.0, 1.0, 1.0 / 256), (1.0, 16.0 / 256, 1.0 / 256), (0.0625, 0.0625, 0.0625)])
def test_a_crowd_costs_no_multiple_of_a_uniform_deposit(box):
    # 10^6 particles in a sheet, in 16 rows of one plane, in a ball: the same passes
    # over the particles and the grid, and no tile whose work grows with its
    # particles.  (The walk over particles took 5 to 13 times the uniform one's time.)
    import torch

    announce("deposit crowds: time", box)
    shape = (256, 256, 256)
    gen = torch.Generator(device="cuda").manual_seed(1)
    uniform = torch.rand((10**6, 3), dtype=torch.float64, device="cuda", generator=gen)
    crowd = 0.4 + uniform * torch.tensor(box, dtype=torch.float64, device="cuda")
    _times(shape, uniform, 3)
    assert _times(shape, crowd) <= 2.5 * _times(shape, uniform)


def test_a_refused_deposit_is_quick():
    # every position bad: all get one key, whose one run is not to be summed before
    # the deposit is refused (it took 70 times a good deposit's time)
    import torch

    announce("deposit: all positions bad")
    shape, n = (256, 256, 256), 10**6
    good = torch.rand((n, 3), dtype=torch.float64, device="cuda")
    bad = torch.full((n, 3), float("nan"), dtype=torch.float64, device="cuda")
    h = P.poisson_create(shape, (1.0, 1.0, 1.0))
    out = torch.full(shape, 7.0, dtype=torch.float64, device="cuda")
    ts = []
    try:
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            with pytest.raises(P.PoissonError) as e:
                P.poisson_deposit(h, bad, None, out)
            ts.append(time.perf_counter() - t)
            assert e.value.code == P.POISSON_EDOMAIN
        assert bool((out == 7.0).all())
    finally:
        P.poisson_destroy(h)
    assert sorted(ts)[2] <= 2.0 * _times(shape, good)
