"""The residual sweeps (P1 and the fused outer residual) on grids of more tiles
than the chip holds at once, where they march along z: every row length from 16
on, planes that do not fill the last tile, rows of whole waves and others, both
boundary conditions and operators.  The solution's residual is measured by the
oracle, so a wrong residual anywhere shows; the norm that the first evaluation
reports is compared with the oracle's."""
import math

import numpy as np
import pytest

import oracle
from gpu_helpers import announce, dev, host
from paper_1601_05448_amd import inputs
from paper_1601_05448_amd import poisson as P

pytestmark = pytest.mark.gpu
TWO_PI = 2.0 * math.pi

# (nz, ny, nx), walls, coef, weight
CASES = [
    ((192, 384, 16), 0, 0, 0), ((96, 512, 24), 1, 0, 0), ((128, 384, 32), 0, 1, 0), ((96, 384, 48), 1, 0, 1),
    ((128, 192, 64), 0, 0, 0), ((96, 192, 96), 0, 0, 0), ((96, 96, 128), 1, 1, 1), ((12, 512, 192), 0, 0, 1),
    ((12, 256, 256), 1, 0, 0), ((12, 256, 384), 0, 0, 0), ((12, 192, 512), 0, 1, 0), ((12, 48, 768), 1, 0, 0),
    ((24, 32, 1024), 0, 0, 0), ((4, 96, 768), 0, 0, 0), ((6, 96, 1024), 1, 1, 0),
]


@pytest.mark.parametrize("shape,walls,coef,weight", CASES)
@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
def test_marched_residual(shape, walls, coef, weight, precision):
    announce("marched residual", shape, walls, coef, weight, precision)
    nz, ny, nx = shape
    h = TWO_PI / min(shape)
    prob = inputs.small_problem(shape=shape, lengths=(nx * h, ny * h, nz * h), ratio=3.0, kmax=2.0)
    b = prob.b - prob.b.mean()
    p0 = 0.1 * np.random.default_rng(1).standard_normal(shape) * h * h
    with P.Solver(shape, prob.lengths, precision=precision, coef=coef, weight=weight, bc_x=walls) as s:
        p = dev(p0)
        st = s.solve(dev(prob.rho), dev(prob.b), p, 1e-10)
        hist = s.history()
    assert st["code"] == P.POISSON_OK, st
    want0 = oracle.residual(prob.rho, prob.b, p0, prob.lengths, coef, bcx=walls)
    # the same sums in another order: relative rounding of sums of squares
    assert abs(hist[0] - want0["r_norm"] / np.linalg.norm(b)) <= 1e-12 * hist[0]
    got = oracle.residual(prob.rho, prob.b, host(p), prob.lengths, coef, bcx=walls)
    assert got["rel"] <= 1e-10 * (1 + 1e-3), got["rel"]
