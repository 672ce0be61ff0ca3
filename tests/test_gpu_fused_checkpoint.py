"""Checkpoints after several steps fused in one launch: every byte is that of
single steps, the sites that pad the last tile of 256 included."""
import pytest
import torch

import helpers as H
from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu


# 12 steps end in a fused launch, 13 on most boxes in a single step
@pytest.mark.parametrize("steps", [12, 13])
@pytest.mark.parametrize("box", [(100, 100), (7, 13), (256, 1), (255, 1), (1001, 601)])
@pytest.mark.parametrize("storage,arith,mode", [("f64", "fp64", "closed"), ("f32", "mixed", "closed"),
                                                ("f16dev", "fp64", "closed"), ("f32", "fp64", "bgk")])
def test_checkpoint_of_fused_steps(gpu, box, storage, arith, mode, steps):
    N = box[0] * box[1]
    f0 = Wk.random_populations(H.textbook_weights(2), N, 0.05, 41, tilt=0.05)
    blobs = []
    for calls in ([steps], [1] * steps):
        sim = gpu.Simulation(2, *box, 1, rho0=torch.ones(N, dtype=torch.float64),
                             u0=torch.zeros(2, N, dtype=torch.float64), beta=0.93,
                             storage=storage, fp64=arith, mode=mode)
        sim.set_populations(f0)
        for c in calls:
            sim.step(c)
        blobs.append(sim.export())
        sim.close()
    assert blobs[0][1] == blobs[1][1] == steps
    assert torch.equal(blobs[0][0], blobs[1][0])
