"""The field of a mesh solve at row lengths and output addresses that do and do
not allow 16-byte stores, against the FP64 oracle (relative L2: 1e-12 FP64,
2e-5 FP32, as for the other mesh solves).  At an address that is only
element-aligned the same bits are expected: each component is one difference
and one product either way."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import poisson_oracle as orc  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"f32": 2e-5, "f64": 1e-12}
NP_DT = {"f32": np.float32, "f64": np.float64}


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("n", [(4, 3, 2), (2, 4, 3), (8, 9, 6), (6, 8, 9), (9, 8, 8), (36, 27, 16), (64, 48, 12)])
def test_field_rows(n, dt):
    from paper_1509_07685_amd import dks
    h = (1e-4, 1.5e-4, 2e-4)
    rho = np.random.default_rng(n[0]).standard_normal((n[2], n[1], n[0])).astype(NP_DT[dt])
    plan = dks.PoissonPlan(n, h, dt)
    dev = torch.from_numpy(rho).cuda()
    _, E = plan.solve_rho(dev)
    buf = torch.full((3 * rho.size + 2,), 7.0, dtype=dev.dtype, device="cuda")
    dks.dks_poisson_solve_rho(plan.handle, dev.data_ptr(), None, buf[1:].data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    _, ref = orc.solve_rho(rho.astype(np.float64), h)
    got = E.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) <= TOL[dt] * np.linalg.norm(ref)
    assert torch.equal(buf[1:-1].view_as(E), E)
    assert float(buf[0]) == 7.0 and float(buf[-1]) == 7.0
