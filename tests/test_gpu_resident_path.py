"""Which solves run on the resident PCG kernel, by the route the library reports: without it a comparison of the
resident kernel with the strip kernel passes where both sides ran the same one.  For each resident route the iterate
is compared with the strip kernel's (plain launches, check_every = 1): 60 iterations, rounding 60 x 1.1e-16 x
sqrt(kappa) with kappa 3e4, 1.2e-12; tolerance 1e-11."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_06824_amd import gapsolve as G  # noqa: E402
from paper_2511_06824_amd.solver import JointGapSolver  # noqa: E402

R, L = G.GAP_PCG_PATH_RESIDENT, G.GAP_PCG_PATH_LAUNCHES
GLOBAL, PER = G.GAP_SCALARS_GLOBAL, G.GAP_SCALARS_PER_COND


def log(msg):
    print(msg, flush=True)


def solver_of(nt, nz, n_cond):
    case = synth.textured_case(nt, nz, 3)
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, case.delta, n_cond)
    return s


@pytest.mark.parametrize("nt,nz,n_cond,path,kw", [
    (150, 61, 9, R, dict()),
    (150, 61, 9, R, dict(strategy=G.GAP_STRATEGY_ASYNC)),
    (150, 61, 9, R, dict(precond=G.GAP_PRECOND_JACOBI)),
    (150, 61, 9, R, dict(graph=False)),
    (150, 61, 9, R, dict(graph=False, check_every=4)),
    (150, 61, 1, R, dict(eps=1e-10)),
    (150, 61, 1, R, dict(eps=1e-10, scalars=PER, strategy=G.GAP_STRATEGY_ASYNC)),
    (260, 704, 9, R, dict()),
    (260, 705, 9, L, dict()),
    (150, 61, 9, L, dict(graph=False, check_every=3)),
    (150, 61, 9, L, dict(scalars=PER)),
    (150, 61, 1, L, dict(eps=1e-8)),
    (150, 61, 9, L, dict(neumann=2)),
    (150, 61, 9, L, dict(precond=G.GAP_PRECOND_ASSOR1)),
    (150, 61, 9, L, dict(iteration=G.GAP_ITERATION_ONE_LAUNCH))])
def test_route_of_a_solve(nt, nz, n_cond, path, kw):
    log(f"case: {nt} x {nz} x {n_cond}, {kw}")
    s = solver_of(nt, nz, n_cond)
    kw = dict(dict(omega=1.6, eps=1e-10, max_iter=60, raise_on_error=False), **kw)
    assert G.gap_pcg_path(s.handle) == G.GAP_PCG_PATH_NONE
    _, i = s.solve(**kw)
    p = s.pressure().clone()
    assert G.gap_pcg_path(s.handle) == path
    if path == R:
        _, j = s.solve(**dict(kw, graph=False, check_every=1))
        assert G.gap_pcg_path(s.handle) == L
        q = s.pressure()
        assert i.iterations == j.iterations and i.status == j.status
        assert max(float((a - b).norm() / b.norm()) for a, b in zip(p, q)) <= 1e-11
    s.close()


def test_route_of_the_adjoint_solves():
    log("case: 150 x 61 x 1, adjoint Jacobian, vector-Jacobian product, base and adjoint systems together")
    s = solver_of(150, 61, 1)
    kw = dict(omega=1.6, eps=1e-10)
    s.solve(**kw)
    assert G.gap_pcg_path(s.handle) == R
    s.jacobian_adjoint(w=np.array([1.0, -0.5, 20.0, 30.0]), **kw)      # one system
    assert G.gap_pcg_path(s.handle) == R
    s.jacobian_adjoint(**kw)                                            # a recurrence for each of four
    assert G.gap_pcg_path(s.handle) == L
    s.solve_with_adjoint(**kw)
    assert G.gap_pcg_path(s.handle) == L
    s.close()


def warm_solver(nt, nz):
    """A solver, its solution, and a function that starts every condition k from solution * (1 + rel[k])."""
    s = solver_of(nt, nz, 9)
    s.solve(omega=1.6, eps=1e-11)
    exact = s.pressure().clone()

    def start(rel):
        rel = torch.tensor(rel, dtype=torch.float64, device="cuda:0")
        s.pressure().copy_(exact * (1.0 + rel.view(9, 1, 1)))
    return s, exact, start


@pytest.mark.parametrize("nt,nz", [(64, 32), (150, 61), (400, 360)])
@pytest.mark.parametrize("max_iter", [100000, 20])
def test_record_of_a_solve_whose_first_condition_freezes_first(nt, nz, max_iter):
    """Another workgroup than that of condition 0 ends the solve: the iterations and status it records stand."""
    log(f"case: {nt} x {nz} x 9, asynchronous test, condition 0 starts near its solution, at most {max_iter} iterations")
    s, exact, start = warm_solver(nt, nz)
    kw = dict(omega=1.6, eps=1e-8, strategy=G.GAP_STRATEGY_ASYNC, warm_start=True, max_iter=max_iter, raise_on_error=False)
    for k in range(6):
        rel = [1e-9 if c == 0 else 10.0 ** -((c + k) % 3) for c in range(9)]
        start(rel)
        _, j = s.solve(graph=False, check_every=1, **kw)
        q = s.pressure().clone()
        for more in (dict(), dict(graph=False, check_every=5)):
            start(rel)
            _, i = s.solve(**kw, **more)
            assert G.gap_pcg_path(s.handle) == R
            assert i.iterations == j.iterations > 0 and i.status == j.status
            assert i.status == (G.GAP_OK if max_iter > 20 else G.GAP_ENOCONV)
            assert max(float((a - b).norm() / b.norm()) for a, b in zip(s.pressure(), q)) <= 1e-9
    s.close()


@pytest.mark.parametrize("nt,nz", [(64, 32), (150, 61), (400, 360)])
def test_conditions_that_freeze_one_after_another(nt, nz):
    """No workgroup is left waiting for words that others have overwritten, which it would do for two seconds
    before the solve is given up.  A joint recurrence from which conditions drop out can break down (64 x 32, the strip
    kernel alike): the residuals are held to the tolerance where the strip kernel converges."""
    log(f"case: {nt} x {nz} x 9, conditions frozen at different passes")
    s, exact, start = warm_solver(nt, nz)
    kw = dict(omega=1.6, eps=1e-8, strategy=G.GAP_STRATEGY_ASYNC, warm_start=True, raise_on_error=False)
    converged = 0
    for rep in range(20):
        rel = [10.0 ** -((k + rep) % 9 / 2) for k in range(9)]
        start(rel)
        _, i = s.solve(**kw)
        assert G.gap_pcg_path(s.handle) == R
        p = s.pressure().clone()
        start(rel)
        _, j = s.solve(graph=False, check_every=1, **kw)
        if j.status == G.GAP_OK:
            converged += 1
            assert i.status == G.GAP_OK and max(i.rel_residual_cond[:9]) <= 1e-8
            assert max(float((a - b).norm() / b.norm()) for a, b in zip(p, exact)) <= 1e-5
    assert converged >= 10
    s.close()


def test_a_warm_start_allocates_nothing():
    """The handle holds what gap_grid_bytes says, also after a warm-started solve, on a handle of nine conditions
    that solves one."""
    log("case: 512 x 256 x 9 and x 1, device memory across the first warm start")
    for n_cond in (9, 1):
        s = solver_of(512, 256, n_cond)
        kw = dict(omega=1.6, eps=1e-10)
        s.solve(**kw)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        s.solve(warm_start=True, **kw)
        assert G.gap_pcg_path(s.handle) == R
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free
        s.close()


@pytest.mark.parametrize("n_cond,kw", [(9, dict()), (9, dict(warm_start=True)), (1, dict(warm_start=True)),
                                       (9, dict(warm_start=True, graph=False, check_every=5)),
                                       (9, dict(warm_start=True, strategy=G.GAP_STRATEGY_ASYNC))])
def test_a_solve_that_gives_the_resident_kernel_up(n_cond, kw):
    """With no time to wait the first look at words not yet published ends the attempt: the solve starts again from
    the same guess on the strip kernel, with its bits, and the handle does not try again until told to."""
    log(f"case: 150 x 61 x {n_cond}, {kw}")
    s = solver_of(150, 61, n_cond)
    kw = dict(dict(omega=1.6, eps=1e-9), **kw)
    s.solve(omega=1.6, eps=1e-3)
    guess = s.pressure().clone()

    def solve():
        s.pressure().copy_(guess)
        _, i = s.solve(**kw)
        return s.pressure().clone(), i.iterations, G.gap_pcg_path(s.handle)

    G.gap_set_resident_wait(s.handle, 0.0)
    p, n, path = solve()
    assert path == L
    G.gap_set_resident_wait(s.handle, 1e-12)
    for expected in (G.GAP_PCG_PATH_GAVE_UP, L):
        q, m, path = solve()
        assert path == expected and m == n and torch.equal(p, q)
    G.gap_set_resident_wait(s.handle, 2.0)
    q, m, path = solve()
    assert path == R and m == n and float((p - q).norm() / p.norm()) <= 1e-9
    for bad in (-1.0, float("nan"), float("inf")):
        with pytest.raises(G.GapError) as ei:
            G.gap_set_resident_wait(s.handle, bad)
        assert ei.value.status == G.GAP_EINVAL
    s.close()


def test_kernel_timing_measures_the_resident_kernel():
    """With timing a solve takes the route it takes without, and its passes are faster than strip launches (at this
    size 8 us against 22)."""
    log("case: 512 x 256 x 9, kernel timing")
    s = solver_of(512, 256, 9)
    kw = dict(omega=1.6, eps=1e-9)
    average = []
    for wait in (2.0, 0.0):
        G.gap_set_resident_wait(s.handle, wait)
        s.solve(**kw)
        G.gap_kernel_timing(s.handle, 1)
        _, i = s.solve(**kw)
        G.gap_kernel_timing(s.handle, 0)
        assert G.gap_pcg_path(s.handle) == (R if wait else L)
        n, ms = G.gap_kernel_stats(s.handle, G.GAP_KERNEL_PCG_STRIPS)
        assert n == i.iterations + 1 if wait else n > i.iterations
        average.append(1e3 * ms / n)
    log(f"  us per pass {average}")
    assert average[0] < 0.75 * average[1]
    s.close()


def test_the_tuner_times_the_strip_kernel():
    """Also where solves run on the resident kernel, which has nothing to tune: the time is that of the strip
    kernel's launches (22 us at this size; the resident kernel's passes take 8)."""
    log("case: 512 x 256 x 9, autotuner")
    s = solver_of(512, 256, 9)
    kw = dict(omega=1.6, eps=1e-9)
    cfg, us = s.tune(iterations=40, **kw)
    assert G.gap_pcg_path(s.handle) == L
    s.solve(**kw)
    assert G.gap_pcg_path(s.handle) == R
    G.gap_set_resident_wait(s.handle, 0.0)
    s.solve(**kw)
    G.gap_kernel_timing(s.handle, 1)
    s.solve(**kw)
    G.gap_kernel_timing(s.handle, 0)
    n, ms = G.gap_kernel_stats(s.handle, G.GAP_KERNEL_PCG_STRIPS)
    log(f"  tuned {cfg['wg_per_cu_w']} workgroups per CU, {us:.1f} us; in a solve {1e3 * ms / n:.1f} us")
    assert 0.7 < us / (1e3 * ms / n) < 1.4
    s.close()


def test_resident_solves_beside_strip_solves_and_a_batch():
    """Resident solves on one stream while a strip solve that fills the chip and then a batch run on another: they
    wait for room on the device, do not give up, and have the bits they have alone."""
    log("case: 512 x 256 x 9 resident, beside 1024 x 512 x 9 strips and a batch of three")
    import threading
    s, big = solver_of(512, 256, 9), solver_of(1024, 512, 9)
    kw = dict(omega=1.6, eps=1e-10)
    _, i = s.solve(**kw)
    alone = s.pressure().clone()
    big.solve(**kw)
    assert G.gap_pcg_path(big.handle) == L
    big_alone = big.pressure().clone()
    torch.cuda.synchronize()
    done, got, wrong = threading.Event(), [], []

    def strips():
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                big.solve(**kw)
                torch.cuda.current_stream().synchronize()
                if not torch.equal(big.pressure(), big_alone):
                    wrong.append("strips")
            members = [solver_of(nt, nz, 9) for nt, nz in ((128, 64), (300, 200), (512, 256))]
            b = G.gap_batch_create()
            st = torch.cuda.current_stream().cuda_stream
            ids = [G.gap_batch_add(b, m.handle, m.options(**kw), m.p.data_ptr(), st) for m in members]
            left = set(ids)
            for _ in range(200):
                G.gap_batch_step(b, 32, True, st)
                for k in G.gap_batch_poll(b):
                    G.gap_batch_remove(b, k, st)
                    left.discard(k)
                if not left:
                    break
            torch.cuda.current_stream().synchronize()
            d = float((members[2].pressure() - alone).norm() / alone.norm())
            if not d <= 1e-9:
                wrong.append(f"batch {d}")
            G.gap_batch_destroy(b)
            for m in members:
                m.close()
        done.set()

    def resident():
        with torch.cuda.stream(torch.cuda.Stream()):
            while not done.is_set() and len(got) < 400:
                _, k = s.solve(**kw)
                torch.cuda.current_stream().synchronize()
                got.append((G.gap_pcg_path(s.handle), k.iterations, torch.equal(s.pressure(), alone)))

    threads = [threading.Thread(target=f) for f in (strips, resident)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    log(f"  {len(got)} resident solves beside the others")
    assert done.is_set() and not wrong
    assert got and all(g == (R, i.iterations, True) for g in got)
    s.close()
    big.close()
