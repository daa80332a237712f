"""A solve takes the fused y, z and y sweeps alone and the single ones in a batch
where the batch makes the launch too large: the same bits, also where the single
sweeps run their wide line groups (32768 lines of 16).  And the fused launch where
it has fewer blocks than columns, so that a block takes several."""
import numpy as np
import pytest

from gpu_helpers import announce, dev, host
from paper_1601_05448_amd import poisson as P

pytestmark = pytest.mark.gpu

SHAPES = [(64, 16, 1024), (16, 64, 1024), (16, 16, 1024), (48, 48, 512)]


def _problem(shape, seed):
    rng = np.random.default_rng(seed)
    rho, b = dev(rng.uniform(1.0, 1.6, shape)), rng.standard_normal(shape)
    return rho, dev(b - b.mean())


@pytest.mark.parametrize("bc", [P.POISSON_BC_PERIODIC, P.POISSON_BC_WALLS_X])
@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_and_single_sweeps_same_bits(shape, precision, bc):
    announce("planes: wide line groups", shape, precision, bc)
    rho, b = _problem(shape, sum(shape))
    h = P.poisson_create(shape, (1.0, 2.0, 1.5), precision=precision, bc_x=bc, max_iter=6)
    try:
        outs = []
        for timed in (0, 2, 3):
            P.poisson_kernel_timer(h, timed, precision == P.POISSON_FP32_REFINE)
            p = dev(np.zeros(shape))
            P.poisson_solve(h, rho, b, p, 1e-14)  # runs into its cap
            outs.append(host(p))
        assert P.poisson_kernel_timer_read(h)[1] > 0
    finally:
        P.poisson_destroy(h)
    assert np.abs(outs[0]).max() > 0.0
    assert np.array_equal(outs[0], outs[1])
    assert np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("precision", [P.POISSON_FP64, P.POISSON_FP32_REFINE])
def test_a_block_takes_several_columns(precision):
    # 512 columns beside requests 64 times smaller: the large request's sweeps get one
    # block on each of half the CUs
    from paper_1601_05448_amd import serve

    announce("planes: several columns per block", precision)
    shapes = [(16, 16, 1024)] + [(16, 16, 16)] * 6
    probs = [_problem(sh, 900 + k) for k, sh in enumerate(shapes)]
    alone, jobs = [], []
    for k, (sh, (rho, b)) in enumerate(zip(shapes, probs)):
        with P.Solver(sh, (1.0, 1.0, 1.0), precision=precision) as s:
            p = dev(np.zeros(sh))
            assert s.solve(rho, b, p, 1e-9)["code"] == P.POISSON_OK
            alone.append(host(p))
        jobs.append(serve.Job(arrival_s=0.0, shape=sh, lengths=(1.0, 1.0, 1.0), rho=rho, b=b, p=dev(np.zeros(sh)), tol=1e-9,
                              tag=k))
    with serve.Server(1 << 30, 16, precision=precision) as s:
        res = serve.replay(s, jobs, realtime=False)
    assert len(res.outcomes) == len(jobs)
    for o in res.outcomes:
        assert np.array_equal(host(o.job.p), alone[o.job.tag]), o.job.tag
