"""Bisection on the power sums, every lattice: each site's alpha against the
stop window with the oracle's G, and its populations against the collision with
that alpha on the oracle's equilibrium."""
import numpy as np
import pytest

import helpers as H
from paper_1904_00866_amd import workloads as Wk
from test_gpu_root_power_sums import EPS, SHAPES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lat", [2, 3, 19])
@pytest.mark.parametrize("eps,far", [(5e-3, 0.0), (0.016, 0.0), (0.035, 0.0), (0.035, 0.02)])
def test_bisection_window_and_collision(gpu, orc, lat, eps, far):
    """-tol <= G(alpha) <= 0 up to the rounding of two sums of Q non-negative terms
    of size D (2 Q eps D, doubled), or alpha = alpha_max with G <= 0 there.  New
    populations to 100 eps (1 + alpha) (f + f^eq): the Q-term moments and the
    equilibrium's few roundings."""
    shape = SHAPES[lat]
    N, D = int(np.prod(shape)), H.dim(lat)
    W = H.textbook_weights(lat)
    f0 = Wk.random_populations(W, N, eps, 700 + lat, tilt=eps / 4)
    if far:
        wild = Wk.random_populations(W, N, 0.6, 701, tilt=0.2)
        pick = np.random.default_rng(702).random(N) < far
        f0 = np.ascontiguousarray(np.where(pick[None, :], wild, f0))
    beta, tol = 0.9, 1e-13
    sim = gpu.Simulation(lat, *shape, rho0=np.ones(N), u0=np.zeros((D, N)), storage="f64",
                         beta=beta, mode="bisect", root_max_iter=200, root_tol=tol,
                         diag=gpu.DIAG_ALPHA)
    sim.set_populations(f0)
    sim.step(1)
    ag = sim.alpha_field().cpu().numpy()
    fg = sim.gather(np.arange(N), 1).cpu().numpy()
    sim.close()
    feq = np.empty_like(f0)
    at_max = 0
    for s in range(N):
        rho, u = orc.moments_site(lat, f0[:, s])
        feq[:, s] = orc.equilibrium(lat, rho, u)
        slack = 1e-16 + 4 * len(W) * EPS * abs(orc.G(lat, f0[:, s], 1.0))
        g = orc.G(lat, f0[:, s], ag[s])
        if -tol - slack <= g <= slack:
            continue
        amax = orc.alpha_max(lat, f0[:, s], feq[:, s])
        assert abs(ag[s] - amax) <= 1e-9 * amax and g <= slack, (s, ag[s], amax, g)
        at_max += 1
    assert at_max < N // 4
    want = f0 + ag * beta * (feq - f0)
    assert np.all(np.abs(fg - want) <= 100 * EPS * (1 + ag) * (f0 + feq))
