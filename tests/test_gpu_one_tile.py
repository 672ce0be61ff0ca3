"""One tile per workgroup (few workgroups, no counts recorded) against four:
the same bits at the edges of tiles, workgroups and the dispatch's line."""
import numpy as np
import pytest
import torch

import helpers as H
from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu

# edges of a tile (256) and of a four-tile workgroup (1024), rows of whole
# blocks, and both sides of the largest one-tile grids: 768 workgroups of 1024
# sites with 4-byte storage, 2304 with 2-byte
SMALL = [(1, 1), (255, 1), (256, 1), (257, 1), (341, 3), (64, 16), (205, 5), (1024, 3)]


def _pair(gpu, nx, ny, mode, storage, arith, f0):
    N = nx * ny
    out = []
    for diag in (0, gpu.DIAG_COUNTS):
        sim = gpu.Simulation(2, nx, ny, 1, rho0=np.ones(N), u0=np.zeros((2, N)), beta=0.92,
                             mode=mode, storage=storage, fp64=arith, diag=diag)
        sim.set_populations(f0)
        sim.step(1)
        out.append(sim.populations())
        sim.close()
    return out


@pytest.mark.parametrize("box", SMALL)
@pytest.mark.parametrize("mode,arith", [("closed", "fp64"), ("closed", "mixed"), ("newton", "fp64"),
                                        ("secant", "fp64"), ("bgk", "fp64")])
@pytest.mark.parametrize("storage", ["f32", "f32dev", "f16dev"])
def test_one_tile_equals_four(gpu, box, mode, arith, storage):
    N = box[0] * box[1]
    near = Wk.random_populations(H.textbook_weights(2), N, 0.02, 11, tilt=0.05,
                                 log_uniform_eps=True)
    far = Wk.random_populations(H.textbook_weights(2), N, 0.6, 12, tilt=0.2)
    f0 = np.where(np.random.default_rng(13).random(N)[None, :] < 0.1, far, near)
    a, b = _pair(gpu, *box, mode, storage, arith, f0)
    assert torch.equal(a, b)


@pytest.mark.parametrize("nx,ny,storage", [(1024, 767, "f32"), (1024, 769, "f32"),
                                           (1001, 785, "f32"), (1024, 2305, "f16dev"),
                                           (1536, 1535, "f16dev")])
def test_one_tile_line(gpu, nx, ny, storage):
    N = nx * ny
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    W = torch.tensor(H.textbook_weights(2), device="cuda")[:, None]
    f0 = W * (1.0 + 0.02 * torch.rand(9, N, dtype=torch.float64, device="cuda", generator=g))
    a, b = _pair(gpu, nx, ny, "closed", storage, "fp64", f0)
    assert torch.equal(a, b)
