"""L^+ through every shape of the y and z sweeps: wide and narrow line groups,
ragged last groups, the register kernels at 256 and 512 and the shapes that
replace them on small grids, each against the oracle with the bounds of
test_gpu_solver (lap_pinv: 1e-12 of the largest value in FP64; FP32: four times
u (2 + 2 sum log2 N) ||q|| over the smallest eigenvalue)."""
import math

import numpy as np
import pytest

import oracle
from gpu_helpers import announce, dev, host
from paper_1601_05448_amd import poisson as P

pytestmark = pytest.mark.gpu
TWO_PI = 2.0 * math.pi

# (nz, ny, nx): the y sweep has nx/2 nz lines, the z sweep nx/2 ny; 512 groups or
# more of the wide shape select it
SHAPES = [
    (512, 96, 96), (96, 512, 96),      # wide groups along y (96) and z (96), 512 lines narrow
    (96, 192, 192), (192, 128, 128),   # wide 192, 128
    (256, 24, 96), (24, 256, 96),      # 256 lines in few groups (no register kernel)
    (384, 6, 768), (6, 384, 768),      # 384 lines in few groups
    (768, 4, 48), (4, 768, 12),        # ragged last groups: 96, 48 and 24 lines
    (1024, 8, 24), (8, 1024, 24),
    (6, 12, 1024), (12, 4, 6), (4, 6, 24),  # single-stage lengths 4, 6, 12
    (32, 512, 32), (16, 48, 24),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
def test_lap_pinv_line_shapes(shape, precision):
    announce("line shapes", shape, precision)
    L = (TWO_PI, 2.5, 4.0)
    q = np.random.default_rng(sum(shape) + 5).standard_normal(shape) + 0.7
    want = oracle.lap_pinv(q, L)
    h = P.poisson_create(shape, L, precision=precision)
    try:
        out = dev(np.zeros(shape))
        (P.poisson_lap_pinv if precision == P.POISSON_FP64 else P.poisson_lap_pinv_fp32)(h, dev(q), out)
    finally:
        P.poisson_destroy(h)
    off = np.max(np.abs(host(out) - want))
    if precision == P.POISSON_FP64:
        assert off <= 1e-12 * np.max(np.abs(want)), shape
    else:
        nz, ny, nx = shape
        lam = min(4.0 * math.sin(math.pi / n) ** 2 * (n / length) ** 2 for n, length in zip((nx, ny, nz), L))
        passes = 2 + 2 * sum(math.log2(n) for n in shape)
        assert off <= 4 * 2.0**-24 * passes * np.linalg.norm(q - q.mean()) / lam, shape


def test_lap_pinv_fp32_thin_cells():
    """Cells 1e6 times longer in x and y than in z, a 48-cell line along z: the
    FP32 inverse symbols span 13 decades."""
    announce("thin cells")
    shape, L = (48, 12, 24), (24e6, 12e6, 48.0)
    q = np.random.default_rng(3).standard_normal(shape)
    q -= q.mean(axis=0, keepdims=True)  # only modes with a z wavenumber: the others are 1e12 larger
    want = oracle.lap_pinv(q, L)
    h = P.poisson_create(shape, L, precision=P.POISSON_FP32_REFINE)
    try:
        out = dev(np.zeros(shape))
        P.poisson_lap_pinv_fp32(h, dev(q), out)
    finally:
        P.poisson_destroy(h)
    got = host(out)
    assert np.all(np.isfinite(got))
    got = got - got.mean(axis=0, keepdims=True)  # rounding puts a little into the large modes
    lam = 4.0 * math.sin(math.pi / 48) ** 2
    bound = 4 * 2.0**-24 * (2 + 2 * sum(math.log2(n) for n in shape)) * np.linalg.norm(q) / lam
    # the z-constant modes' rounding, up to 1e12 / (4 sin^2(pi/24)) times larger,
    # is removed above up to its own FP32 rounding
    stray = np.max(np.abs(host(out))) * 2.0**-23 * 4
    assert np.max(np.abs(got - want)) <= bound + stray
