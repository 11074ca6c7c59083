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

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

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
