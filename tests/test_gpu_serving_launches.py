"""The server counts the kernel launches it makes."""
import pytest
import torch

from paper_1904_00866_amd import workloads as Wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [(64, dict(storage="f32", beta=0.99)),
                                  (48, dict(storage="f16dev", beta=0.99, mode="newton"))])
def test_launches_of_one_request(gpu, n, kw):
    """Rounds of 20, 20 and 7 steps; steps of the first kind share launches."""
    rho, u = Wk.shear_layer(n)
    with gpu.Server(64 << 20, max_active=4, round_steps=20, stream=torch.cuda.Stream()) as srv:
        srv.wait(srv.submit(2, n, n, rho0=rho, u0=u, nsteps=47, **kw), 60.0)
        st = srv.stats()
    cfg = gpu.make_config("d2q9", n, n, **kw)
    want = sum(gpu.batch_launches([cfg], [k]) for k in (20, 20, 7))
    assert st["rounds"] == 3 and st["launches"] == want
    assert want == 47 if "mode" in kw else want < 47
