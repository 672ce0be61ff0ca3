"""Fused steps of the types and boxes that take them beyond the small boxes, on
states with sites far from equilibrium (every tier of the rare phase)."""
import pytest
import torch

import helpers as H
from test_gpu_fused import SMALL, _compare, _state

pytestmark = pytest.mark.gpu

# type and boxes where the dispatch fuses steps (checked): each geometry that it
# takes for the type, ragged and in whole blocks, and thin boxes
F64, F32, DEV, F16 = "f64", "f32", "f32dev", "f16dev"
LARGE = [((F64, "fp64", "closed"), [(480, 480), (1001, 601), (64, 4099)]),
         ((F64, "fp64", "bgk"), [(480, 480), (1001, 601), (33, 9001)]),
         ((F32, "fp64", "bgk"), [(633, 632), (1024, 513), (64, 8192)]),
         ((DEV, "fp64", "bgk"), [(633, 632), (1001, 601)]),
         ((F32, "fp64", "closed"), [(1001, 901), (1024, 1024)]),
         ((F32, "fp32", "closed"), [(480, 480), (1001, 601), (32, 32768)]),
         ((F32, "mixed", "closed"), [(480, 480), (1001, 601), (1450, 1447)]),
         ((DEV, "mixed", "closed"), [(480, 480), (1001, 601), (1450, 1447)]),
         ((F16, "fp64", "bgk"), [(1450, 1447)]),
         ((F16, "mixed", "closed"), [(64, 4096), (480, 480), (1450, 1447)])]


@pytest.mark.parametrize("kind,box", [(k, b) for k, bs in LARGE for b in bs])
def test_fused_far_states(gpu, kind, box):
    nx, ny = box
    storage, arith, mode = kind
    cfg = gpu.make_config("d2q9", nx, ny, storage=storage, fp64=arith, mode=mode)
    assert gpu.batch_launches([cfg], [4]) < 4
    N = nx * ny
    g = torch.Generator(device="cuda").manual_seed(N)

    def rnd(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)

    W = torch.tensor(H.textbook_weights(2), device="cuda")[:, None]
    near = 1.0 + 0.05 * rnd(9, N) ** 4
    far = torch.exp(1.6 * (rnd(9, N) - 0.5))  # max|x_i| of about 0.1 to 1.5
    f0 = W * torch.where(rnd(1, N) < 0.04, far, near)
    _compare(gpu, nx, ny, kind, f0, 4)


@pytest.mark.parametrize("kind", [(DEV, "mixed", "closed"), (DEV, "fp64", "bgk"),
                                  (DEV, "fp32", "closed")])
@pytest.mark.parametrize("box", SMALL)
def test_fused_small_boxes_of_deviations(gpu, box, kind):
    _compare(gpu, *box, kind, _state(box[0] * box[1], 37), 7)
