"""Small grids, whose y, z and y sweeps run as one launch on whole planes: L^+
against the oracle over the lengths that have it (bounds of test_gpu_line_shapes:
FP64 1e-12 of the largest value; FP32 four times u (2 + 2 sum log2 N) ||q|| over
the smallest eigenvalue), and whole solves against the same solve with its y
sweeps timed, which run one by one: the same bits."""
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


def _exact_x_mode(want, q, L):
    """`want` with its part that depends on x alone replaced by the exact one
    between walls: u'' = f has the fluxes h sum f.  (The oracle's tridiagonal
    solve of this singular mode is off by up to 1.7e-14 on these inputs, 1.4e-12
    of the largest value, measured against these sums in extended precision.)"""
    ld = np.longdouble
    f = q.astype(ld).mean(axis=(0, 1))
    f -= f.mean()
    h = ld(L[0]) / q.shape[2]
    u = np.concatenate([[ld(0)], np.cumsum(np.cumsum(f)[:-1] * h * h)])
    u -= u.mean()
    return (want + (u - want.astype(ld).mean(axis=(0, 1)))).astype(np.float64)


LENGTHS = (16, 24, 32, 48, 64)


@pytest.mark.parametrize("bc", [P.POISSON_BC_PERIODIC, P.POISSON_BC_WALLS_X])
@pytest.mark.parametrize("nz", LENGTHS)
@pytest.mark.parametrize("ny", LENGTHS)
def test_lap_pinv_planes(ny, nz, bc):
    announce("planes", nz, ny, bc)
    rng = np.random.default_rng(64 * ny + nz)
    for nx in (4, 24):
        shape, L = (nz, ny, nx), (2.0, 2.5, 4.0)
        q = rng.standard_normal(shape) + 0.7
        walls = bc == P.POISSON_BC_WALLS_X
        want = oracle.lap_pinv(q, L, bcx=oracle.BC_WALLS_X if walls else oracle.BC_PERIODIC)
        if walls:
            want = _exact_x_mode(want, q, L)
        h = P.poisson_create(shape, L, precision=P.POISSON_FP32_REFINE, bc_x=bc)
        try:
            out, out32 = dev(np.zeros(shape)), dev(np.zeros(shape))
            P.poisson_lap_pinv(h, dev(q), out)
            P.poisson_lap_pinv_fp32(h, dev(q), out32)
        finally:
            P.poisson_destroy(h)
        assert np.max(np.abs(host(out) - want)) <= 1e-12 * np.max(np.abs(want)), shape
        # walls: the x modes are cos(pi k (i + 1/2) / nx), half the periodic angle
        lam = min([4.0 * math.sin(math.pi / n) ** 2 * (n / length) ** 2 for n, length in zip((ny, nz), L[1:])] +
                  [4.0 * math.sin(math.pi / (2 * nx if walls else nx)) ** 2 * (nx / L[0]) ** 2])
        passes = 2 + 2 * sum(math.log2(n) for n in shape)
        bound = 4 * 2.0**-24 * passes * np.linalg.norm(q - q.mean()) / lam
        assert np.max(np.abs(host(out32) - want)) <= bound, shape


@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
@pytest.mark.parametrize("shape", [(32, 32, 32), (48, 48, 24), (16, 64, 48), (24, 16, 256), (64, 64, 64)] +
                         [(nz, ny, 16) for nz in LENGTHS for ny in LENGTHS])
def test_solve_same_bits_as_single_sweeps(shape, precision):
    announce("planes: solve", shape, precision)
    rng = np.random.default_rng(sum(shape))
    rho, b = dev(rng.uniform(1.0, 4.0, shape)), rng.standard_normal(shape)
    b = dev(b - b.mean())
    h = P.poisson_create(shape, (1.0, 2.0, 1.5), precision=precision)
    try:
        outs = []
        for timed in (False, True):
            if timed:
                P.poisson_kernel_timer(h, 2, precision == P.POISSON_FP32_REFINE)
            p = dev(np.zeros(shape))
            P.poisson_solve(h, rho, b, p, 1e-9)
            outs.append(host(p))
        _, launches = P.poisson_kernel_timer_read(h)
        assert launches > 0
    finally:
        P.poisson_destroy(h)
    assert np.array_equal(outs[0], outs[1])
