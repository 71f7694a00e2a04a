"""The direct deposit of small solves where many particles share nodes: one
cell, a few cells, bunches a whole number of the combining blocks (16 x 8 x 8
nodes) apart, a broad bunch, particles outside the mesh, one particle.

Its node totals are exact integers, so the density has to be bit for bit that
of the order-independent deposit, which bins and is held against the oracle
elsewhere; the out-of-mesh counts are equal too."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TORCH = {"f32": torch.float32, "f64": torch.float64}
N, H = (72, 36, 48), 1e-4


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


def positions(shape, num, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(num)
    r = torch.randn(3, num, generator=g, device="cuda", dtype=TORCH[dt]) * H
    if shape == "bunches":          # three blocks apart on every axis
        k = torch.arange(num, device="cuda") % 3 - 1
        r = 0.3 * r + torch.tensor([[16.0], [8.0], [8.0]], device="cuda", dtype=TORCH[dt]) * H * k
        return r
    return r * {"cell": 0.05, "cells": 0.6, "broad": 8.0, "outside": 30.0}[shape]


@pytest.mark.parametrize("shape", ["cell", "cells", "bunches", "broad", "outside"])
@pytest.mark.parametrize("dt,scheme,num", [
    ("f32", "cic", 32768), ("f32", "cic", 127), ("f32", "ngp", 200_001), ("f32", "tsc", 9709), ("f32", "ngp", 1),
    ("f64", "cic", 32767), ("f64", "cic", 129), ("f64", "ngp", 32767), ("f64", "tsc", 9709), ("f64", "tsc", 1)])
def test_density_equals_the_order_independent_one(dt, scheme, num, shape):
    pos = positions(shape, num, dt)
    plan = dks().PoissonPlan(N, (H,) * 3, dt, scheme=scheme)
    for _ in range(2):
        rho, cnt = plan.deposit(*pos, 1.0)
    plan.set_deterministic(True)
    ref, rcnt = plan.deposit(*pos, 1.0)
    torch.cuda.synchronize()
    assert int(cnt.item()) == int(rcnt.item())
    assert torch.equal(rho, ref)
