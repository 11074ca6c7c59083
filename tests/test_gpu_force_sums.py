"""Rounding error of the pressure force where nearly all of it cancels: the mean pressure and a third harmonic around
the ring leave no force, so what is returned is the error of the sums.

Tolerance: ring by ring a thread meets at most 16 columns spread over the ring, whose running sum stays near the size
of a term (rms 1.2 of the largest pressure for 8 columns).  N additions and N products, each off by 2^-53 / sqrt(3) of that,
add at random to 1.1e-16 sqrt(N); the tolerance is three times that, of N times the largest term, on the root mean
square over conditions and components.  Sums that cancel only between workgroups are off by 5 times the tolerance or
more (1.6e-18 against 3.2e-19 at 2048 x 512, where the ring order leaves 4e-20).  The last case has more columns than
the LDS keeps."""

import math

import numpy as np
import pytest

import oracle
import synth
from conftest import gap_of, texture_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2511_06824_amd import gapsolve as G  # noqa: E402
from paper_2511_06824_amd.solver import JointGapSolver  # noqa: E402


@pytest.mark.parametrize("nt,nz,n_cond", [(2048, 512, 9), (2048, 256, 9), (4000, 130, 9)])
def test_pressures_that_cancel_around_the_ring(nt, nz, n_cond):
    print(nt, nz, n_cond, flush=True)
    case = synth.smooth_case(nt, nz, 2)
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, case.delta, n_cond)
    dth, dz = 2.0 * math.pi / nt, case.L / nz
    theta = np.array([(i + 0.5) * dth for i in range(nt)])
    z = (np.arange(nz) + 0.5) * dz
    p = np.stack([case.p_in * (1.0 - 0.99 * z / case.L)[:, None] + 0.4 * case.p_in *
                  np.sin(3 * theta + 0.7 * k) * np.sin(math.pi * z / case.L)[:, None] for k in range(n_cond)])
    dev = torch.from_numpy(p.ravel()).to("cuda:0")
    got = s.integrate_split(p=dev).cpu().numpy()[:, :4] / (case.R * dth * dz)
    s.close()
    cos = np.array([math.cos(t) for t in theta]).astype(np.longdouble)
    sin = np.array([math.sin(t) for t in theta]).astype(np.longdouble)
    zr = (z - 0.5 * case.L).astype(np.longdouble)[:, None]
    err = []
    for k in range(n_cond):
        a, b = -p[k].astype(np.longdouble) * cos, -p[k].astype(np.longdouble) * sin
        exact = [a.sum(), b.sum(), -(zr * b).sum(), (zr * a).sum()]
        err += [float(got[k, q] - exact[q]) / (case.p_in * nt * nz * (1.0 if q < 2 else case.L / 2)) for q in range(4)]
    rms = math.sqrt(np.mean(np.square(err)))
    print(f"  rms {rms:.1e}, largest {max(map(abs, err)):.1e}", flush=True)
    assert rms <= 3.3e-16 / math.sqrt(nt * nz)


@pytest.mark.parametrize("nt,nz,n_cond", [(3, 2, 9), (5, 65536, 9), (513, 1500, 9), (3072, 40, 9), (3073, 40, 9), (9000, 3, 1)])
def test_both_kernels_match_the_oracle(nt, nz, n_cond):
    """Rings that the LDS keeps and longer ones, grids of two and three rows, chunks of more rows than are prepared
    at once (64; 65536 rows make chunks of 580).  Tolerance as for sums of up to 1e6 terms whose sizes add to a few times
    the force, in trees and runs below 1000 terms: 1000 x 2^-53 x 5 = 6e-13, so 2e-12."""
    print(nt, nz, n_cond, flush=True)
    case = synth.smooth_case(nt, nz, 5)
    gap = gap_of(case)
    s = JointGapSolver.from_case(case, max_cond=9)
    s.assemble(case.e, case.edot, case.delta, n_cond)
    theta = (np.arange(nt) + 0.5) * (2 * np.pi / nt)
    rng = np.random.default_rng(nt)
    p = 1e6 * (0.8 + 0.6 * np.cos(theta + 0.3) + 0.1 * rng.random((n_cond, nz, nt)))
    dev = torch.from_numpy(p.ravel()).to("cuda:0")
    F = s.integrate(G.GAP_CAVITATION_CLAMP, 4e5, p=dev).cpu().numpy()
    split = s.integrate_split(G.GAP_CAVITATION_CLAMP, 4e5, p=dev).cpu().numpy()
    s.close()
    conds = oracle.conditions(case.e, case.edot, case.delta)
    for k in sorted({0, n_cond - 1}):
        F_r = oracle.forces_for_condition(gap, conds[k][0], p[k].ravel(), texture_of(case), cavitation="clamp", p_cav=4e5)
        for sl in (slice(0, 2), slice(2, 4)):
            largest = np.abs(F_r[sl]).max()
            total = split[k, sl] + split[k, 4 + sl.start:4 + sl.stop]
            assert np.abs(F[k, sl] - F_r[sl]).max() <= 2e-12 * largest
            assert np.abs(total - F_r[sl]).max() <= 2e-12 * largest
