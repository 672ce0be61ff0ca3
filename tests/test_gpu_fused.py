"""Several steps fused in one launch against single steps: the same bits, on
boxes smaller than a region, at the edges of tiles, rows of whole blocks and
on both sides of the dispatch's lines, near and far from equilibrium."""
import numpy as np
import pytest
import torch

import helpers as H
from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu

KINDS = [("f64", "fp64", "closed"), ("f32", "fp64", "closed"), ("f32dev", "fp64", "closed"),
         ("f16dev", "fp64", "closed"), ("f32", "mixed", "closed"), ("f16dev", "mixed", "closed"),
         ("f32", "fp32", "closed"), ("f16dev", "fp32", "closed"), ("f64", "fp64", "bgk"),
         ("f32", "fp64", "bgk"), ("f16dev", "fp64", "bgk")]
# up to six steps per launch: interiors of 6 .. 14 of a 16 x 16 region
SMALL = [(1, 1), (2, 5), (6, 6), (7, 13), (16, 16), (64, 14), (97, 101), (192, 130)]
# beyond 1024 regions of three steps: the large geometries, ragged and not,
# around the 400,000 sites where some types change theirs
LARGE = [(480, 480), (633, 632), (1024, 513), (1001, 601), (1450, 1447)]


def _state(N, seed):
    W = H.textbook_weights(2)
    near = Wk.random_populations(W, N, 0.02, seed, tilt=0.05, log_uniform_eps=True)
    far = Wk.random_populations(W, N, 0.6, seed + 1, tilt=0.2)
    return np.where(np.random.default_rng(seed + 2).random(N)[None, :] < 0.05, far, near)


def _compare(gpu, nx, ny, kind, f0, steps):
    N = nx * ny
    storage, arith, mode = kind
    kw = dict(rho0=torch.ones(N, dtype=torch.float64), u0=torch.zeros(2, N, dtype=torch.float64),
              beta=0.93, storage=storage, fp64=arith, mode=mode)
    out = []
    for calls in ([steps], [1] * steps):
        sim = gpu.Simulation(2, nx, ny, 1, **kw)
        sim.set_populations(f0)
        for c in calls:
            sim.step(c)
        assert sim.t == steps
        out.append((sim.populations(), *sim.moments()))
        sim.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("box", SMALL)
def test_fused_small_boxes(gpu, box, kind):
    """Seven steps: six and one, five and two, ... by the box."""
    _compare(gpu, *box, kind, _state(box[0] * box[1], 31), 7)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("box", LARGE)
def test_fused_large_boxes(gpu, box, kind):
    N = box[0] * box[1]
    g = torch.Generator(device="cuda").manual_seed(N)
    W = torch.tensor(H.textbook_weights(2), device="cuda")[:, None]
    f0 = W * (1.0 + 0.05 * torch.rand(9, N, dtype=torch.float64, device="cuda", generator=g) ** 4)
    _compare(gpu, *box, kind, f0, 4)


@pytest.mark.parametrize("diag", [2, 7])
def test_fused_then_recorded(gpu, diag):
    """The recording last step after fused ones: the diagnostics of single steps;
    a batch of boxes with other step counts gives each box's own bits."""
    boxes, steps = [(70, 33), (16, 50), (130, 64)], [9, 4, 17]
    sims = []
    for r in range(2):
        sims.append([])
        for (nx, ny) in boxes:
            N = nx * ny
            rho, u = Wk.random_velocity_field(2, N, 0.1, seed=nx)
            sims[r].append(gpu.Simulation(2, nx, ny, 1, rho0=rho, u0=u, beta=0.95, diag=diag))
    gpu.step_batch(sims[0], steps)
    for s, n in zip(sims[1], steps):
        for _ in range(n):
            s.step(1)
    for a, b in zip(*sims):
        assert a.t == b.t and torch.equal(a.populations(), b.populations())
        assert a.stats() == b.stats()
        if diag & 1:
            assert torch.equal(a.alpha_field(), b.alpha_field())
        a.close()
        b.close()


@pytest.mark.parametrize("n", [2, 4, 6, 10, 12, 26])
@pytest.mark.parametrize("nx,ny,storage", [(96, 80, "f32"), (520, 500, "f64")])
def test_fused_under_capture(gpu, nx, ny, storage, n):
    """A captured call of an even number of steps, replayed with other work
    between the replays, against eager steps: the state returns to the buffer
    it began in, as it does after single steps."""
    rho, u = Wk.random_velocity_field(2, nx * ny, 0.05, seed=9)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        kw = dict(rho0=rho, u0=u, beta=0.95, storage=storage, stream=stream)
        sim = gpu.Simulation(2, nx, ny, 1, **kw)
        ref = gpu.Simulation(2, nx, ny, 1, **kw)
        sim.step(n)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(n)
        for _ in range(3):
            graph.replay()
            torch.ones(1000, device="cuda").sum()
            stream.synchronize()
        ref.step(4 * n)
        assert torch.equal(sim.populations(), ref.populations())
        sim.close()
        ref.close()
