"""The root solvers on the power sums: sites on either side of the tiers'
bounds on max|x_i| (8.5e-3, 0.025, 0.05), whole wavefronts within them and
wavefronts mixed with sites far beyond."""
import numpy as np
import pytest

import helpers as H
from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu

SHAPES = {2: (70, 37, 1), 3: (19, 13, 11), 19: (19, 13, 11)}
EPS = 2.0 ** -52


@pytest.mark.parametrize("lat", [2, 3, 19])
@pytest.mark.parametrize("eps,far", [(5e-3, 0.0), (0.016, 0.0), (0.035, 0.0), (0.035, 0.02)])
@pytest.mark.parametrize("mode", ["newton", "bisect"])
def test_root_power_sums(gpu, orc, lat, eps, far, mode):
    """One FP64 step against the oracle: populations within 1e-13 (1e-12 with
    far sites), Newton's alpha within 1e-12 plus the oracle's own conditioning
    10 eps / |2 - alpha| (its phi carry eps |x|, and |2 - alpha| <= 2 |x| / 3);
    bisection's alphas inside its window."""
    shape = SHAPES[lat]
    N = int(np.prod(shape))
    W = H.textbook_weights(lat)
    f0 = Wk.random_populations(W, N, eps, 600 + lat, tilt=eps / 4)
    if far:
        wild = Wk.random_populations(W, N, 0.6, 601, tilt=0.2)
        pick = np.random.default_rng(602).random(N) < far
        f0 = np.ascontiguousarray(np.where(pick[None, :], wild, f0))
    D = H.dim(lat)
    sim = gpu.Simulation(lat, *shape, rho0=np.ones(N), u0=np.zeros((D, N)), storage="f64",
                         beta=0.9, mode=mode, root_max_iter=200, diag=gpu.DIAG_ALPHA)
    sim.set_populations(f0)
    sim.step(1)
    fg, ag = sim.populations().cpu().numpy(), sim.alpha_field().cpu().numpy()
    sim.close()
    kw = dict(q=19) if lat == 19 else {}
    cfg = orc.Config(D=D, nx=shape[0], ny=shape[1], nz=shape[2], beta=0.9, mode=mode,
                     root_max_iter=200, **kw)
    fo, ao, _ = orc.step(cfg, f0, want_alpha=True, want_diag=True)
    if mode == "newton":
        assert np.max(np.abs(fg - fo) / np.abs(fo)) <= (1e-12 if far else 1e-13)
        tol = (1e-11 if far else 1e-12) + 10 * EPS / np.maximum(np.abs(2 - ao), 1e-9)
        assert np.all(np.abs(ag - ao) <= tol)
    elif lat != 19:
        for s in np.nonzero(np.abs(ag - ao) > 1e-14)[0][:400]:
            g = orc.G(D, f0[:, s], ag[s])
            assert -1e-13 - 1e-16 <= g <= 1e-16, (s, g)
