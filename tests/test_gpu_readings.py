"""The readings of the state (populations, moments, gathers) and its setting on
boxes of every load form, and the diagnostics reduction on both sides of its
one-launch limit, against values formed from the populations in FP64."""
import numpy as np
import pytest
import torch

import helpers as H

pytestmark = pytest.mark.gpu

# rows of whole 64-site blocks, one row short of a workgroup, ragged, one site
BOXES = {1: [(64, 1, 1), (832, 1, 1), (301, 1, 1), (1, 1, 1)],
         2: [(64, 5, 1), (192, 7, 1), (65, 3, 1), (1, 1, 1)],
         3: [(64, 3, 2), (128, 2, 3), (9, 7, 5), (1, 1, 1)],
         19: [(64, 3, 2), (128, 2, 3), (9, 7, 5), (1, 1, 1)]}


@pytest.mark.parametrize("lat", [1, 2, 3, 19])
@pytest.mark.parametrize("box", range(4))
def test_set_and_read_populations(gpu, lat, box):
    """FP64 storage: set_populations then populations gives the same bits; the
    gather of every site too; rho and u within the rounding of their Q-term
    sums (Q eps relative to the terms) of numpy's."""
    shape = BOXES[lat][box]
    N = int(np.prod(shape))
    c = H.abi_velocities(lat)[:, :H.dim(lat)]
    Q, D = c.shape
    f0 = H.textbook_weights(lat)[:, None] * \
        (1.0 + 0.2 * np.random.default_rng(70 + lat).standard_normal((Q, N)))
    sim = gpu.Simulation(lat, *shape, rho0=np.ones(N), u0=np.zeros((D, N)), storage="f64")
    sim.set_populations(f0)
    assert np.array_equal(sim.populations().cpu().numpy(), f0)
    assert np.array_equal(sim.gather(np.arange(N)).cpu().numpy(), f0)
    rho, u = (t.cpu().numpy() for t in sim.moments())
    sim.close()
    eps = Q * 2.0 ** -52
    assert np.all(np.abs(rho - f0.sum(0)) <= eps * np.abs(f0).sum(0))
    j = c.T.astype(float) @ f0
    assert np.all(np.abs(u * rho - j) <= 2 * eps * np.abs(f0).sum(0) + 4e-16 * np.abs(j))


def test_moments_of_nonfinite_populations(gpu):
    """One infinite and one NaN population: their sites' velocity is NaN in
    every component, the other sites are untouched."""
    shape = (70, 5, 1)
    N = 350
    f0 = H.textbook_weights(2)[:, None] * np.ones((9, N))
    f0[1, 17] = np.inf
    f0[3, 200] = np.nan
    sim = gpu.Simulation(2, *shape, rho0=np.ones(N), u0=np.zeros((2, N)), storage="f64")
    sim.set_populations(f0)
    rho, u = (t.cpu().numpy() for t in sim.moments())
    sim.close()
    assert np.isinf(rho[17]) and np.isnan(rho[200])
    assert np.isnan(u[:, [17, 200]]).all()
    ok = np.setdiff1d(np.arange(N), [17, 200])
    assert np.isfinite(rho[ok]).all() and np.isfinite(u[:, ok]).all()


@pytest.mark.parametrize("nx,ny", [(1024, 1024),   # 4096 records: one launch
                                   (1031, 1021),   # 4112: two, the last chunk short
                                   (1600, 1483)])  # 9272 records
def test_reduction_of_many_records(gpu, nx, ny):
    """Counts equal those of the recorded alpha field; sum rho, rho u and H
    within N eps of the sums of their absolute terms; a second reading gives
    the same bits."""
    N = nx * ny
    g = torch.Generator(device="cuda").manual_seed(nx)
    W = torch.tensor(H.textbook_weights(2), device="cuda")[:, None]
    f0 = W * (1.0 + 0.01 * (2.0 * torch.rand(9, N, dtype=torch.float64, device="cuda",
                                             generator=g) - 1.0))
    sim = gpu.Simulation(2, nx, ny, 1, rho0=torch.ones(N, dtype=torch.float64),
                         u0=torch.zeros(2, N, dtype=torch.float64), storage="f64", beta=0.9,
                         diag=gpu.DIAG_ALPHA | gpu.DIAG_COUNTS | gpu.DIAG_SUMS)
    sim.set_populations(f0)
    sim.step(1)
    st, again, a = sim.stats(), sim.stats(), sim.alpha_field()
    sim.close()
    assert st == again
    assert st["n_alpha_lt2"] == int((a < 2.0).sum())
    assert st["n_sites"] == N and st["n_nonfinite"] == 0
    assert st["alpha_min"] == float(a.min().float())
    assert st["alpha_max"] == float(a.max().float())
    tol = N * 2.0 ** -52
    assert abs(st["sum_rho"] - float(f0.sum())) <= tol * float(f0.sum())
    c = torch.tensor(H.abi_velocities(2)[:, :2].T.astype(float), device="cuda")
    j = (c @ f0).sum(1).cpu().numpy()
    assert np.all(np.abs(np.array(st["sum_j"][:2]) - j) <= tol * float(f0.sum()))
    h = f0 * torch.log(f0 / W)
    assert abs(st["sum_H"] - float(h.sum())) <= tol * float(h.abs().sum())
