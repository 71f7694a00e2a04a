"""Mesh solves on both sides of the sizes at which the y pass stores past the
caches, against the FP64 oracle: relative L2 1e-12 FP64, 2e-5 FP32, as for the
other mesh solves.  Solved twice with another solve between, so that a value
left in a cache would show."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import poisson_oracle as orc  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"f32": 2e-5, "f64": 1e-12}
NP_DT = {"f32": np.float32, "f64": np.float64}


@pytest.mark.parametrize("dt,n", [("f64", (96, 108, 192)), ("f64", (96, 128, 192)), ("f32", (128, 256, 108)),
                                  ("f32", (256, 128, 128)), ("f64", (144, 144, 128))])
def test_large_mesh(dt, n):
    from paper_1509_07685_amd import dks
    h = (1e-4, 1.5e-4, 2e-4)
    rng = np.random.default_rng(n[1])
    rho = rng.standard_normal((n[2], n[1], n[0])).astype(NP_DT[dt])
    plan = dks.PoissonPlan(n, h, dt)
    dev = torch.from_numpy(rho).cuda()
    first, _ = plan.solve_rho(dev, want_E=False)
    plan.solve_rho(dev.flip(0).contiguous(), want_E=False)
    phi, _ = plan.solve_rho(dev, want_E=False)
    torch.cuda.synchronize()
    ref = orc.solve_rho(rho.astype(np.float64), h)[0][1:-1, 1:-1, 1:-1]
    assert torch.equal(first, phi)
    assert np.linalg.norm(phi.cpu().numpy() - ref) <= TOL[dt] * np.linalg.norm(ref)
