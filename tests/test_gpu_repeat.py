"""Repeated refinement solves of one problem, launched one by one and from graphs:
the same bits, the same counts of steps and sweeps.  (An update or a decision that
took part of its state from after the launch's last block had changed it would
differ from run to run.)"""
import numpy as np
import pytest

from gpu_helpers import announce, dev, host
from paper_1601_05448_amd import poisson as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 12, 12), (32, 32, 32), (96, 48, 96), (128, 128, 128)])
def test_refinement_repeats_its_bits(shape):
    announce("repeated refinement", shape)
    rng = np.random.default_rng(sum(shape))
    rho, b = dev(rng.uniform(1.0, 4.0, shape)), rng.standard_normal(shape)
    b = dev(b - b.mean())
    first = None
    for graphs in (0, 1):
        with P.Solver(shape, (1.0, 2.0, 1.5), precision=P.POISSON_FP32_REFINE, use_graphs=graphs) as s:
            for _ in range(6):
                p = dev(np.zeros(shape))
                st = s.solve(rho, b, p, 1e-10)
                got = (host(p), st["iters"], st["outer_iters"], st["p1_sweeps"], list(s.history()))
                if first is None:
                    first = got
                assert np.array_equal(got[0], first[0])
                assert got[1:] == first[1:]
