"""Only the last step of a call records diagnostics: what can be read after
step(n) equals what n calls of one step leave."""
import numpy as np
import pytest
import torch

from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("diag", [1, 2, 3, 7])
@pytest.mark.parametrize("lattice,shape", [("d2q9", (70, 33, 1)), ("d3q27", (12, 10, 9))])
def test_step_n_equals_n_steps(gpu, lattice, shape, diag):
    N, D = int(np.prod(shape)), 2 if lattice == "d2q9" else 3
    rho, u = Wk.random_velocity_field(D, N, 0.1, seed=3)
    sims = [gpu.Simulation(lattice, *shape, rho0=rho, u0=u, beta=0.95, diag=diag)
            for _ in range(3)]
    sims[0].step(5)
    for _ in range(5):
        sims[1].step(1)
    gpu.step_batch([sims[2], sims[0]], [5, 0])
    out = [(s.populations(), s.alpha_field() if diag & 1 else None,
            s.stats() if diag & 2 else None) for s in sims]
    for s in sims:
        s.close()
    for f, a, st in out[1:]:
        assert torch.equal(f, out[0][0])
        assert a is None or torch.equal(a, out[0][1])
        assert st == out[0][2]
