"""More simulations than share a launch, of sizes whose groups fuse differently:
each has the bits, the time and the diagnostics that it has alone."""
import numpy as np
import pytest
import torch

from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,arith", [("f32", "fp64"), ("f16dev", "mixed"), ("f64", "fp64")])
def test_groups_equal_alone(gpu, storage, arith):
    boxes = [(64, 64)] * 9 + [(37, 91), (200, 130), (5, 700)] + [(128, 128)] * 6 + \
            [(16, 16), (301, 77), (1, 900)]
    steps = [12, 7, 30, 12, 0, 1, 12, 5, 30, 12, 30, 12, 12, 9, 30, 30, 2, 12, 30, 12, 9]
    sims = [[], []]
    for k, (nx, ny) in enumerate(boxes):
        rho, u = Wk.random_velocity_field(2, nx * ny, 0.1, seed=k)
        for r in sims:
            r.append(gpu.Simulation(2, nx, ny, 1, rho0=rho, u0=u, beta=0.95, storage=storage,
                                    fp64=arith, diag=(0, 2, 7)[k % 3]))
    gpu.step_batch(sims[0], steps)
    for s, n in zip(sims[1], steps):
        s.step(n)
    for k, (a, b) in enumerate(zip(*sims)):
        assert a.t == b.t == steps[k]
        assert torch.equal(a.export()[0], b.export()[0]), k
        if steps[k] and k % 3:
            assert a.stats() == b.stats(), k
        if steps[k] and k % 3 == 2:
            assert torch.equal(a.alpha_field(), b.alpha_field()), k
        a.close()
        b.close()
