"""Which solves deposit and gather without binning, read off the names of the
kernels that a solve runs, at both sides of the rules' lines."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TORCH = {"f32": torch.float32, "f64": torch.float64}


def kernels(n, dt, scheme, num):
    from paper_1509_07685_amd import dks
    g = torch.Generator(device="cuda")
    g.manual_seed(num)
    pos = [torch.rand(num, generator=g, device="cuda", dtype=TORCH[dt]) * 1e-4 for _ in range(3)]
    plan = dks.PoissonPlan(n, (1e-4,) * 3, dt, scheme=scheme)
    dks.dks_timing_enable(1)
    try:
        plan.solve_particles(*pos, 1e-15)
        torch.cuda.synchronize()
        return set(dks.dks_timing_read())
    finally:
        dks.dks_timing_enable(0)


@pytest.mark.parametrize("n,dt,direct", [
    ((256, 256, 256), "f32", True),      # 2^24 nodes
    ((256, 256, 288), "f32", False),
    ((256, 256, 288), "f64", True),      # totals as wide as the weights
])
def test_small_deposits_on_large_meshes(n, dt, direct):
    assert ("bin_count" not in kernels(n, dt, "cic", 1000)) == direct


@pytest.mark.parametrize("dt,scheme,num", [
    ("f32", "cic", 1 << 18), ("f32", "ngp", 1 << 18), ("f64", "cic", 1 << 18),
    ("f32", "tsc", 1 << 17), ("f64", "tsc", 3 << 15),      # 162 reads of phi a particle
])
def test_gathers_in_the_callers_order(dt, scheme, num):
    assert "unsort" not in kernels((32, 24, 36), dt, scheme, num)
    assert "unsort" in kernels((32, 24, 36), dt, scheme, num + 1)
