"""Grouped-row loads: with 4- and 2-byte storage, D1Q3 and D2Q9 boxes whose
x-rows hold whole groups of four 256-site tiles load them with the first tile's
offsets.  Launches of few workgroups take one tile each unless they record
counts, so these simulations record them."""
import numpy as np
import pytest
import torch

import helpers as H
from paper_1904_00866_amd import workloads as Wk
from test_gpu_parity import GROUP_SHAPES, _ocfg, _random_state, _sim, _storage_rounding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", GROUP_SHAPES)
@pytest.mark.parametrize("storage", ["f32", "f32dev", "f16dev"])
@pytest.mark.parametrize("mode", ["closed", "bgk", "mixed"])
def test_grouped_rows_against_the_oracle(gpu, orc, shape, storage, mode):
    """One step from the decoded stored state, every site (both wraps included),
    to one output rounding with FP64 site arithmetic; mixed arithmetic to 2e-6
    relative more, as the other mixed one-step tests."""
    D = 1 if shape[1] == 1 else 2
    f0 = _random_state(D, int(np.prod(shape)), seed=960 + 10 * D + len(storage) + len(mode),
                       eps=0.02, tilt=0.05)
    arith, amode = ("mixed", "closed") if mode == "mixed" else (True, mode)
    sim = _sim(gpu, D, shape, f0, storage=storage, beta=0.97, mode=amode, fp64=arith,
               diag=gpu.DIAG_COUNTS)
    fq = sim.populations().cpu().numpy()
    sim.step(1)
    fg = sim.populations().cpu().numpy()
    sim.close()
    fo, _, _ = orc.step(_ocfg(orc, D, shape, beta=0.97, mode=amode), fq)
    tol = _storage_rounding(storage, fo, H.textbook_weights(D)[:, None])
    if mode == "mixed":
        tol = tol + 2e-6 * np.abs(fo)
    assert np.all(np.abs(fg - fo) <= tol)


@pytest.mark.parametrize("nx", [1, 255, 257, 1024, 2048, 3000, 5120])
@pytest.mark.parametrize("storage,mode,arith", [("f32", "closed", "fp64"), ("f32", "newton", "fp64"),
                                                ("f32dev", "closed", "mixed"),
                                                ("f32dev", "bgk", "fp64"),
                                                ("f16dev", "closed", "fp64"),
                                                ("f16dev", "secant", "fp64"),
                                                ("f16dev", "closed", "mixed")])
def test_one_tile_equals_four_d1q3(gpu, nx, storage, mode, arith):
    """D1Q3, a step recorded (four tiles per workgroup) and not (one): the same
    bits, near and far from equilibrium."""
    W = H.textbook_weights(1)
    near = Wk.random_populations(W, nx, 0.02, 21, tilt=0.05, log_uniform_eps=True)
    far = Wk.random_populations(W, nx, 0.6, 22, tilt=0.2)
    f0 = np.where(np.random.default_rng(23).random(nx)[None, :] < 0.1, far, near)
    out = []
    for diag in (0, gpu.DIAG_COUNTS):
        sim = _sim(gpu, 1, (nx, 1, 1), f0, storage=storage, beta=0.92, mode=mode, fp64=arith,
                   diag=diag)
        sim.step(1)
        out.append(sim.export()[0])
        sim.close()
    assert torch.equal(*out)
