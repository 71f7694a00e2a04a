"""Mesh solves on both sides of the 90 MiB from which the y pass stores past
the caches (81, 96 and 97 MiB of spectrum), and a batch that crosses it by its
number of elements, against the FP64 oracle: relative L2 1e-12 FP64, 2e-5 FP32,
as for the other solves.  Solved twice with another solve between, so that a
value left in a cache would show."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import poisson_oracle as orc  # noqa: E402
from paper_1509_07685_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"f32": 2e-5, "f64": 1e-12}
NP_DT = {"f32": np.float32, "f64": np.float64}


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


@pytest.mark.parametrize("dt,n", [("f32", (128, 192, 192)), ("f32", (128, 216, 216)), ("f64", (144, 144, 144))])
def test_large_mesh(dt, n):
    h = (1e-4, 1.5e-4, 2e-4)
    rho = np.random.default_rng(n[1]).standard_normal((n[2], n[1], n[0])).astype(NP_DT[dt])
    plan = dks().PoissonPlan(n, h, dt)
    dev = torch.from_numpy(rho).cuda()
    first, _ = plan.solve_rho(dev, want_E=False)
    plan.solve_rho(dev.flip(0).contiguous(), want_E=False)
    phi, _ = plan.solve_rho(dev, want_E=False)
    torch.cuda.synchronize()
    ref = orc.solve_rho(rho.astype(np.float64), h)[0][1:-1, 1:-1, 1:-1]
    assert torch.equal(first, phi)
    assert np.linalg.norm(phi.cpu().numpy() - ref) <= TOL[dt] * np.linalg.norm(ref)


def test_batch_over_the_line():
    """16 elements of 64 x 96 x 48 FP32 (90 MiB together) against the oracle."""
    n, batch, num = (64, 96, 48), 16, 5000
    plan = dks().PoissonPlan(n, None, "f32")
    sets = [[torch.from_numpy(a).cuda() for a in wl.gaussian_bunch(num, (1e-3, 1e-3, 2e-3), 40 + i, np.float32)]
            for i in range(batch)]
    outs = [[torch.empty_like(p[0]) for _ in range(3)] for p in sets]
    table = dks().particle_set_table([
        {"x": p[0].data_ptr(), "y": p[1].data_ptr(), "z": p[2].data_ptr(), "Ex": o[0].data_ptr(),
         "Ey": o[1].data_ptr(), "Ez": o[2].data_ptr(), "np": num, "q": 1e-14} for p, o in zip(sets, outs)])
    plan.solve_particles_batched(torch.frombuffer(bytearray(table), dtype=torch.uint8).cuda(), batch, num,
                                 plan.batch_scratch(batch, num))
    torch.cuda.synchronize()
    for i in (0, 7, 15):
        x, y, z = (a.cpu().numpy() for a in sets[i])
        ref = orc.solve_particles(x, y, z, 1e-14, n, dtype=np.float32)
        got = torch.stack(outs[i]).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref["E"]) <= TOL["f32"] * np.linalg.norm(ref["E"])
