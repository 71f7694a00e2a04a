"""Binned kernels at particle counts and with options that keep solves off the
direct ones of small solves: the tile search of the deposit and gather at 63,
64 and 4096 tiles, arrays of unaligned positions or outputs, and one tile of
many work items.

Tolerances (relative L2): density 1e-12 FP64 and max(2e-5, 3.5 n 2^-24) FP32
(the cell coordinate's rounding), fields 1e-12 and 2e-5, as for the other
steps.  The tile-ordered step's field is compared with the direct gather's of
the same potential (the order-independent deposit gives both the same bits):
the same interpolation, so far closer than the tolerance."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import poisson_oracle as orc  # noqa: E402
from paper_1509_07685_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"f32": 2e-5, "f64": 1e-12}
NP_DT = {"f32": np.float32, "f64": np.float64}
TORCH = {"f32": torch.float32, "f64": torch.float64}
MESHES = [(108, 144, 16), (64, 64, 64), (1024, 512, 32)]     # 63, 64 and 4096 tiles, and the outside one


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def rho_tol(dt, n):
    return TOL[dt] if dt == "f64" else max(TOL[dt], 3.5 * max(n) * 2.0 ** -24)


def spread(n, h, num, dt):
    g = np.random.default_rng(num + n[0])
    return [(g.uniform(-0.5, 0.5, num) * (n[d] - 1) * 0.999 * h[d]).astype(NP_DT[dt]) for d in range(3)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("deterministic,num", [(False, 40_000), (True, 20_000)])
@pytest.mark.parametrize("n", MESHES)
def test_binned_deposit_of_many_tiles(n, deterministic, num, dt):
    h = (1e-4, 1.2e-4, 0.8e-4)
    pos = spread(n, h, num, dt)
    plan = dks().PoissonPlan(n, h, dt)
    plan.set_deterministic(deterministic)
    rho, cnt = plan.deposit(*[torch.from_numpy(p).cuda() for p in pos], 1.0)
    torch.cuda.synchronize()
    Q, n_out = orc.deposit_cic(*pos, 1.0, n, h, orc.centred_origin(n, h), NP_DT[dt])
    assert int(cnt.item()) == n_out == 0
    assert rel_l2(rho.cpu().numpy().astype(np.float64) * np.prod(h), Q) <= rho_tol(dt, n)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,scheme", [(MESHES[0], "cic"), (MESHES[0], "tsc"), (MESHES[1], "cic"), (MESHES[1], "ngp"),
                                      (MESHES[1], "tsc"), (MESHES[2], "cic")])
def test_binned_gather_of_many_tiles(n, scheme, dt):
    h, num = (1e-4, 1e-4, 1e-4), 30_000
    pos = [torch.from_numpy(p).cuda() for p in spread(n, h, num, dt)]
    plan = dks().PoissonPlan(n, h, dt, scheme=scheme)
    plan.set_deterministic(True)
    E, phi, cnt = plan.solve_particles(*pos, 1e-13, want_phi=True)
    out, Es, phis, cnts, idx = plan.solve_particles_sorted(*pos, 1e-13, want_phi=True, want_index=True)
    torch.cuda.synchronize()
    assert torch.equal(phi, phis) and torch.equal(cnt, cnts)
    i = idx.long()
    for a, b in zip(pos + list(E), list(out) + list(Es)):
        a, b = a.cpu().numpy().astype(np.float64), b[i].cpu().numpy().astype(np.float64)
        assert rel_l2(b, a) <= TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_unaligned_positions_and_outputs_of_a_binned_step(dt):
    """Positions and outputs unaligned each by itself: the scatter's and the
    unsort's element layouts then differ."""
    n, num, q = (48, 48, 48), (1 << 18) + 777, 2e-14
    x, y, z = wl.gaussian_bunch(num, (1e-3, 0.7e-3, 1.3e-3), 91, NP_DT[dt])
    plan = dks().PoissonPlan(n, None, dt)

    def shifted(off, a=None):
        buf = torch.zeros(num + 1, dtype=TORCH[dt], device="cuda")[off:off + num]
        if a is not None:
            buf.copy_(torch.from_numpy(a))
        return buf

    ref = orc.solve_particles(x, y, z, q, n, dtype=NP_DT[dt])
    for off_in, off_out in ((0, 0), (1, 0), (0, 1), (1, 1)):
        out = tuple(shifted(off_out) for _ in range(3)) + (torch.zeros(1, dtype=torch.int64, device="cuda"),)
        plan.solve_particles(*(shifted(off_in, a) for a in (x, y, z)), q, out=out)
        torch.cuda.synchronize()
        assert int(out[3].item()) == 0
        got = torch.stack(out[:3]).cpu().numpy().astype(np.float64)
        assert rel_l2(got, ref["E"]) <= TOL[dt], (off_in, off_out)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_field_of_a_dense_tile_of_many_items(dt):
    n, h, num, q = (48, 48, 48), (1e-4, 1e-4, 1e-4), 300_000, 1e-15
    origin = orc.centred_origin(n, h)
    g = np.random.default_rng(31)
    x, y, z = ((origin[d] + (17.0 + 14.0 * g.random(num)) * h[d]).astype(NP_DT[dt]) for d in range(3))
    E, _, _ = dks().PoissonPlan(n, h, dt).solve_particles(*(torch.from_numpy(a).cuda() for a in (x, y, z)), q)
    torch.cuda.synchronize()
    ref = orc.solve_particles(x, y, z, q, n, h, dtype=NP_DT[dt])
    assert rel_l2(torch.stack(E).cpu().numpy().astype(np.float64), ref["E"]) <= TOL[dt]
