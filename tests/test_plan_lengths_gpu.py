"""Every transform length with compile-time kernels, in each of its roles.

The convolution runs x rows of nx and y and z pencils of 2 ny and 2 nz on
kernels compiled for the length (16 to 512, each 2^a 3^b); the raw transforms
run rows and columns of those lengths likewise.  Here every such length is an
x, a y and a z extent once, against the FP64 oracles, in FP32 and FP64, with
extents beside it whose tiles are ragged.

Tolerances (relative L2 over the whole output), as for the other shapes: phi
and E 2e-5 in FP32 and 1e-12 in FP64; raw transforms 1e-5 and 1e-12 (the unit
roundoff times the passes, at most 27 radix-2 levels, is 2e-6 and 4e-15)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import fft_oracle as fo  # noqa: E402
from oracle import poisson_oracle as orc  # noqa: E402
from paper_1509_07685_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu

POISSON_TOL = {"f32": 2e-5, "f64": 1e-12}
FFT_TOL = {"f32": 1e-5, "f64": 1e-12}
NP_DT = {"f32": np.float32, "f64": np.float64}
RDT = {"f32": torch.float32, "f64": torch.float64}
CDT = {"f32": torch.complex64, "f64": torch.complex128}

SHORT = [16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108]      # mesh extents
LONG = [128, 144, 162, 192, 216, 243, 256]
RAW = SHORT + LONG + [288, 324, 384, 432, 486, 512]                # raw transform lengths


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


def rel_l2(a, b):
    a, b = np.asarray(a).ravel(), np.asarray(b).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


MESHES = [(SHORT[i], SHORT[(i + 4) % 13], SHORT[(i + 8) % 13]) for i in range(13)]
MESHES += [m for n in LONG for m in ((n, 16, 9), (12, n, 16), (16, 12, n))]


@pytest.mark.parametrize("n", MESHES)
def test_mesh_extents(n):
    h = (1e-4, 2e-4, 1.5e-4)
    rho = np.random.default_rng(n[0] + 300 * n[1] + 90000 * n[2]).standard_normal((n[2], n[1], n[0]))
    for dt in ("f64", "f32"):
        r = rho.astype(NP_DT[dt])
        plan = dks().PoissonPlan(n, h, dt)
        phi, E = plan.solve_rho(torch.from_numpy(r).cuda())
        torch.cuda.synchronize()
        phi_ref, E_ref = orc.solve_rho(r.astype(np.float64), h)
        assert rel_l2(phi.cpu().numpy(), phi_ref[1:-1, 1:-1, 1:-1]) <= POISSON_TOL[dt], dt
        assert rel_l2(E.cpu().numpy(), E_ref) <= POISSON_TOL[dt], dt


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rho_at_an_odd_element_offset(dt):
    """A density whose address is not a multiple of a pair of reals."""
    n, h = (48, 18, 16), (1e-4, 1e-4, 1e-4)
    buf = torch.from_numpy(np.random.default_rng(3).standard_normal(48 * 18 * 16 + 1).astype(NP_DT[dt])).cuda()
    rho = buf[1:].view(16, 18, 48)
    phi, _ = dks().PoissonPlan(n, h, dt).solve_rho(rho, want_E=False)
    torch.cuda.synchronize()
    ref, _ = orc.solve_rho(rho.cpu().numpy().astype(np.float64), h)
    assert rel_l2(phi.cpu().numpy(), ref[1:-1, 1:-1, 1:-1]) <= POISSON_TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("nz", SHORT + LONG)
def test_batched_solve_equals_single_solves(nz, dt):
    """Batched solves take the one-shot z kernel, single ones the persistent
    one where it is compiled for the length."""
    n = (18, 16, nz)
    plan = dks().PoissonPlan(n, None, dt)
    sets = [[torch.from_numpy(a).cuda() for a in wl.gaussian_bunch(m, (1e-3, 2e-3, 1e-3), 40 + m, NP_DT[dt])]
            for m in (3000, 4097)]
    outs = [[torch.empty_like(p[0]) for _ in range(3)] for p in sets]
    table = dks().particle_set_table([
        {"x": p[0].data_ptr(), "y": p[1].data_ptr(), "z": p[2].data_ptr(), "Ex": o[0].data_ptr(),
         "Ey": o[1].data_ptr(), "Ez": o[2].data_ptr(), "np": p[0].numel(), "q": 1e-12} for p, o in zip(sets, outs)])
    dev = torch.frombuffer(bytearray(table), dtype=torch.uint8).cuda()
    plan.solve_particles_batched(dev, 2, 5000, plan.batch_scratch(2, 5000))
    torch.cuda.synchronize()
    for p, o in zip(sets, outs):
        E, _, _ = plan.solve_particles(*p, 1e-12)
        torch.cuda.synchronize()
        assert rel_l2(torch.stack(o).cpu().numpy(), torch.stack(E).cpu().numpy()) <= POISSON_TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", RAW)
def test_raw_lengths(n, dt):
    g = np.random.default_rng(n)
    for shape, batch in (((n, 6, 1), 4), ((18, n, 2), 1), ((3, 9, n), 2)):
        nx, ny, nz = shape
        x = torch.from_numpy(g.standard_normal((batch, nz, ny, nx)) + 1j * g.standard_normal((batch, nz, ny, nx)))
        x = x.to(CDT[dt]).cuda()
        plan = dks().FFTPlan(shape, batch, "c2c", dt)
        X, Y = plan.forward(x), plan.inverse(x)
        torch.cuda.synchronize()
        xq = x.cpu().numpy().astype(np.complex128)
        assert rel_l2(X.cpu().numpy(), fo.dft3(xq)) <= FFT_TOL[dt], shape
        assert rel_l2(Y.cpu().numpy(), fo.dft3(xq, inverse=True)) <= FFT_TOL[dt], shape
        r = torch.from_numpy(g.standard_normal((batch, nz, ny, nx))).to(RDT[dt]).cuda()
        plan = dks().FFTPlan(shape, batch, "r2c", dt)
        H = plan.forward(r)
        y = plan.inverse(H)
        torch.cuda.synchronize()
        assert rel_l2(H.cpu().numpy(), fo.rdft3(r.cpu().numpy())) <= FFT_TOL[dt], shape
        assert rel_l2(y.cpu().numpy() / (nx * ny * nz), r.cpu().numpy()) <= FFT_TOL[dt], shape


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,batch", [((256, 256, 128), 1), ((162, 243, 216), 1), ((48, 128, 128), 16)])
def test_raw_wide_column_tiles(n, batch, dt):
    """Arrays of 64 MiB and more run columns of up to 256 elements in wider
    tiles; the last tile of a row or plane may be ragged."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n[0])
    x = torch.randn((batch, n[2], n[1], n[0]), generator=g, dtype=CDT[dt], device="cuda")
    plan = dks().FFTPlan(n, batch, "c2c", dt)
    X = plan.forward(x)
    ref = torch.fft.fftn(x.to(torch.complex128), dim=(1, 2, 3))
    assert float((X - ref).abs().norm() / ref.norm()) <= FFT_TOL[dt]
    y = plan.inverse(X) / (n[0] * n[1] * n[2])
    assert float((y - x).norm() / x.norm()) <= FFT_TOL[dt]
    r = x.real.contiguous()
    plan = dks().FFTPlan(n, batch, "r2c", dt)
    H = plan.forward(r)
    ref = torch.fft.rfftn(r.double(), dim=(1, 2, 3))
    assert float((H - ref).abs().norm() / ref.norm()) <= FFT_TOL[dt]
    assert float((plan.inverse(H) / (n[0] * n[1] * n[2]) - r).norm() / r.norm()) <= FFT_TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_raw_real_rows_at_an_odd_element_offset(dt):
    """Real arrays whose address is not a multiple of a pair of reals."""
    n = (48, 6, 4)
    buf = torch.from_numpy(np.random.default_rng(4).standard_normal(2 * 48 * 24 + 1)).to(RDT[dt]).cuda()
    x = buf[1:].view(2, 4, 6, 48)
    out = torch.zeros_like(buf)[1:].view(2, 4, 6, 48)
    plan = dks().FFTPlan(n, 2, "r2c", dt)
    H = plan.forward(x)
    plan.inverse(H, out=out)
    torch.cuda.synchronize()
    assert rel_l2(H.cpu().numpy(), fo.rdft3(x.cpu().numpy())) <= FFT_TOL[dt]
    assert rel_l2(out.cpu().numpy() / (48 * 24), x.cpu().numpy()) <= FFT_TOL[dt]
