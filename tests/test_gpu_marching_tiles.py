"""The residual sweeps on grids that must march along z: more small tiles than the
chip could hold at once whatever a kernel's registers and LDS are (32 waves per CU),
so that neither precision and neither sweep (P1, the fused outer residual) takes
them.  Every row length that has both kinds of tiles; planes that do not fill the
last flush where a grid can have so many tiles with them (rows of 192 and longer);
both boundary conditions and operators.  Measured as in test_gpu_residual_tiles:
the first norm and the final residual against the oracle's."""
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
    ((256, 768, 16), 1, 0, 0), ((128, 768, 24), 0, 0, 0), ((96, 768, 32), 0, 1, 0), ((64, 768, 48), 1, 0, 1),
    ((48, 768, 64), 0, 0, 0), ((24, 1024, 96), 1, 0, 0), ((24, 768, 128), 0, 1, 1), ((12, 1024, 192), 0, 0, 1),
    ((12, 768, 256), 1, 0, 0), ((24, 384, 256), 0, 0, 0), ((12, 512, 384), 0, 1, 0), ((12, 384, 512), 1, 0, 0),
    ((24, 192, 512), 0, 0, 0),
]


def _small_tile_threads(shape):
    """Threads of all the small tiles: one per column of a row pair and two planes."""
    nz, ny, nx = shape
    return math.ceil(nz / 2) * (ny // 2) * nx


@pytest.mark.parametrize("shape,walls,coef,weight", CASES)
@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
def test_marching_residual(shape, walls, coef, weight, precision):
    import torch

    announce("marching residual", shape, walls, coef, weight, precision)
    assert _small_tile_threads(shape) > torch.cuda.get_device_properties(0).multi_processor_count * 2048
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
