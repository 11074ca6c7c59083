"""GPU tests of the resident PCG kernel (all iterations of a solve in one cooperative launch) at
the sizes where its tiling can go wrong: every tile height, grids that end inside a tile, rings
narrower than a strip or one column past it; with every recurrence and stopping variant.

Oracle of these tests: the launch-per-iteration strip kernel, which a host that reads the record
after every iteration gets (plain launches, check_every = 1) and which the other files hold
against the CPU oracle.  After j iterations both iterates carry rounding of about
j 2^-53 sqrt(kappa) relative: 80 x 1.1e-16 x sqrt(3e4) = 1.5e-12; the tolerance is 1e-11."""

import threading

import numpy as np
import pytest
import torch

import synth
from paper_2511_06824_amd import gapsolve as G
from paper_2511_06824_amd.solver import JointGapSolver

pytestmark = pytest.mark.gpu
TOL = 1e-11


def log(msg):
    print(msg, flush=True)


def solver_of(nt, nz, n_cond, seed=3, kind=synth.textured_case):
    case = kind(nt, nz, seed)
    s = JointGapSolver.from_case(case, max_cond=9 if n_cond > 1 else 1)
    s.assemble(case.e, case.edot, case.delta if n_cond == 9 else None, n_cond)
    return s, case


def solve(s, **kw):
    _, info = s.solve(raise_on_error=False, **kw)
    return s.pressure().clone(), info


def check(s, label, **kw):
    """The strip kernel's iterate, the resident one's, and the same bits with timed launches and in
    blocks of 5 iterations."""
    ref, ri = solve(s, graph=False, check_every=1, **kw)
    p, i = solve(s, **kw)
    d = max(float((p[k] - ref[k]).norm() / ref[k].norm()) for k in range(p.shape[0]))
    log(f"  {label}: iterations {i.iterations} / {ri.iterations}, difference {d:.1e}")
    assert i.iterations == ri.iterations and i.status == ri.status and d <= TOL
    assert abs(i.rel_residual - ri.rel_residual) <= 1e-6 * ri.rel_residual
    for k in range(p.shape[0]):
        assert abs(i.rel_residual_cond[k] - ri.rel_residual_cond[k]) <= 1e-6 * max(ri.rel_residual_cond[k], 1e-300)
    G.gap_kernel_timing(s.handle, 1)
    pt, it = solve(s, **kw)
    G.gap_kernel_timing(s.handle, 0)
    pb, ib = solve(s, graph=False, check_every=5, **kw)
    for q, info in ((pt, it), (pb, ib)):
        assert torch.equal(p, q) and info.iterations == i.iterations and info.rel_residual == i.rel_residual
        assert list(info.rel_residual_cond) == list(i.rel_residual_cond)
    return p, i


# a ring of 260 columns (5 strips) with 9 conditions: the axial sizes at which the tile height
# changes (4 to 32 rows), full and one row into the next tile
@pytest.mark.parametrize("nz", [68, 69, 102, 103, 137, 171, 205, 239, 273, 353, 441, 529, 617, 704])
@pytest.mark.parametrize("precond", [G.GAP_PRECOND_ASSOR2, G.GAP_PRECOND_JACOBI], ids=["assor2", "jacobi"])
def test_every_tile_height_matches_the_strip_kernel(nz, precond):
    log(f"case: 260 x {nz} x 9, preconditioner {precond}")
    s, case = solver_of(260, nz, 9)
    check(s, "80 iterations", omega=1.6, eps=1e-300, max_iter=80, precond=precond)
    s.close()


@pytest.mark.parametrize("nt,nz,n_cond", [(3, 2, 9), (7, 5, 9), (51, 6, 9), (52, 9, 9), (53, 4, 9), (104, 31, 1),
                                          (105, 33, 9), (1000, 16, 9), (2080, 200, 1), (4000, 17, 1), (64, 1000, 1)])
def test_odd_grids_match_the_strip_kernel(nt, nz, n_cond):
    log(f"case: {nt} x {nz} x {n_cond}")
    s, case = solver_of(nt, nz, n_cond, kind=synth.smooth_case)
    for max_iter in (1, 2, 25):
        check(s, f"{max_iter} iterations", omega=1.8, eps=1e-300, max_iter=max_iter)
    s.close()


@pytest.mark.parametrize("scalars", [G.GAP_SCALARS_GLOBAL, G.GAP_SCALARS_PER_COND], ids=["global", "per_cond"])
@pytest.mark.parametrize("strategy", [G.GAP_STRATEGY_SYNC, G.GAP_STRATEGY_ASYNC], ids=["sync", "async"])
@pytest.mark.parametrize("n_cond", [1, 9])
def test_recurrence_and_stopping_variants(scalars, strategy, n_cond):
    """Solves to convergence, cold and warm; conditions that freeze at different iterations (async)."""
    log(f"case: 150 x 61 x {n_cond}, scalars {scalars}, strategy {strategy}")
    s, case = solver_of(150, 61, n_cond)
    kw = dict(omega=1.6, scalars=scalars, strategy=strategy)
    p, i = check(s, "cold", eps=1e-8, **kw)
    assert i.status == G.GAP_OK
    start = p.clone() * 1.01

    def warm(**more):
        s.p.view(-1)[: start.numel()].copy_(start.reshape(-1))
        return solve(s, eps=1e-9, warm_start=True, **kw, **more)

    ref, ri = warm(graph=False, check_every=1)
    q, qi = warm()
    d = float((q - ref).norm() / ref.norm())
    log(f"  warm: iterations {qi.iterations} / {ri.iterations}, difference {d:.1e}")
    assert qi.iterations == ri.iterations and d <= TOL and qi.true_rel_residual <= 1.2e-9
    s.close()


def test_adjoint_systems_that_stop_on_their_own():
    """Base and four adjoint systems (5 conditions on one operator), the adjoint ones at a looser tolerance, so
    that they freeze before the base system ends."""
    log("case: 200 x 80, base + 4 adjoint systems")
    s, case = solver_of(200, 80, 1)
    s.close()
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, None, 1)
    out = []
    for more in (dict(graph=False, check_every=1), dict()):
        p, J, info = s.solve_with_adjoint(omega=1.6, eps=1e-10, eps_adjoint=1e-7, **more)
        out.append((p.clone(), J.clone(), info.iterations))
    assert out[0][2] == out[1][2]
    assert float((out[0][0] - out[1][0]).norm() / out[0][0].norm()) <= TOL
    assert float((out[0][1] - out[1][1]).norm() / out[0][1].norm()) <= 1e-10
    s.close()


@pytest.mark.parametrize("nt,nz", [(64, 32), (150, 61), (700, 300)])
def test_one_condition_solved_to_a_tight_tolerance(nt, nz):
    """One condition, and base + adjoint systems with a recurrence each, to 1e-10: two orders of summation end
    within the error of the solves, about 10 eps in p and lambda (J is linear in lambda)."""
    log(f"case: {nt} x {nz} x 1 and base + 4 adjoint systems, eps 1e-10")
    case = synth.textured_case(nt, nz, 4)
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, None, 1)
    out = []
    for more in (dict(graph=False, check_every=1), dict()):
        p1, i1 = solve(s, omega=1.6, eps=1e-10, **more)
        p, J, info = s.solve_with_adjoint(omega=1.6, eps=1e-10, **more)
        out.append((p1, i1.iterations, p.clone(), J.clone(), info.iterations))
        assert i1.status == G.GAP_OK and i1.true_rel_residual <= 1.2e-10
    (a1, n1, a, Ja, na), (b1, m1, b, Jb, nb) = out
    diffs = [float((x - y).norm() / x.norm()) for x, y in ((a1, b1), (a, b), (Ja, Jb))]
    log(f"  iterations {n1} / {m1} and {na} / {nb}, differences {diffs}")
    assert abs(n1 - m1) <= 1 and abs(na - nb) <= 1
    assert max(diffs) <= 1e-9
    s.close()


def test_two_threads_on_their_own_streams():
    """Two solves at once on two streams give the bits each gives alone."""
    log("case: two threads, 256 x 128 x 9 and 96 x 50 x 9")
    cases = [solver_of(256, 128, 9, 1), solver_of(96, 50, 9, 2)]
    kw = dict(omega=1.6, eps=1e-10)
    alone = [solve(s, **kw) for s, _ in cases]
    got = [[], []]

    def run(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got[k].append(solve(cases[k][0], **kw))
                torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert len(got[k]) == 4
        for p, i in got[k]:
            assert i.iterations == alone[k][1].iterations and torch.equal(p, alone[k][0])
        cases[k][0].close()


def test_recorded_scalars_match_the_strip_kernel():
    log("case: 128 x 64 x 9, recorded alpha and beta")
    s, case = solver_of(128, 64, 9)
    out = []
    for more in (dict(graph=False, check_every=1), dict()):
        G.gap_pcg_history(s.handle, 64)
        solve(s, omega=1.6, eps=1e-300, max_iter=40, **more)
        out.append(G.gap_get_pcg_history(s.handle, 64))
    assert len(out[0][0]) == len(out[1][0]) == 40
    for a, b in zip(*out):
        np.testing.assert_allclose(a, b, rtol=1e-9)
    s.close()
