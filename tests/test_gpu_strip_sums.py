"""Partial sums and scalars at the start of a strip iteration: 1 to several hundred slots a condition (the
rounds of 64 the kernel loads ahead, and those past them), wavefronts with none to three conditions,
GLOBAL and PER_COND scalars, frozen conditions.

Both kernels run the same recurrence; they add in another order.  A sum over a grid of n <= 1.3e6 cells by trees
and rows of at most 150 serial terms is off by at most 200 x 2^-53 = 2e-14 of the sum of its terms' sizes, and alpha
and beta of 6 iterations carry that into the residual norms with a factor below 20 (quotients of sums, z^T A z by
parts): 1e-11 leaves a decade of room."""

import numpy as np
import pytest
import torch

import synth
from paper_2511_06824_amd import gapsolve as G
from paper_2511_06824_amd.solver import JointGapSolver

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.mark.parametrize("scalars,strategy", [(G.GAP_SCALARS_GLOBAL, G.GAP_STRATEGY_SYNC),
                                              (G.GAP_SCALARS_PER_COND, G.GAP_STRATEGY_SYNC),
                                              (G.GAP_SCALARS_PER_COND, G.GAP_STRATEGY_ASYNC)])
@pytest.mark.parametrize("nt,nz,n_cond", [(64, 20, 1), (300, 47, 9), (1024, 256, 1), (2048, 600, 1),
                                          (1000, 800, 9)])
def test_residual_norms_match_the_two_launch_iteration(nt, nz, n_cond, scalars, strategy):
    print(nt, nz, n_cond, scalars, strategy, flush=True)
    case = synth.textured_case(nt, nz, 5)
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, case.delta, n_cond)
    got = []
    for iteration in (G.GAP_ITERATION_STRIPS, G.GAP_ITERATION_TWO_LAUNCH):
        p, info = s.solve(s.options(eps=1e-6, max_iter=6, scalars=scalars, strategy=strategy, iteration=iteration),
                          raise_on_error=False)
        torch.cuda.synchronize()
        got.append((p.cpu().numpy().copy(), info.rel_residual, np.array(info.rel_residual_cond[:n_cond])))
    s.close()
    (p, rel, rel_c), (p2, rel2, rel_c2) = got
    assert abs(rel - rel2) <= TOL * rel2
    assert np.all(np.abs(rel_c - rel_c2) <= TOL * rel_c2)
    assert np.abs(p - p2).max() <= TOL * np.abs(p2).max()
