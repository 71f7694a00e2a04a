"""Real rows of 576 to 1024 points, which run on half-length complex transforms
of three passes, with a last tile of few rows, forward and inverse against the
FP64 DFT oracle: at an even and at an odd element offset (pairs of reals in one
load, or two).  Relative L2 1e-12 FP64, 1e-5 FP32, as for the other lengths."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import fft_oracle as fo  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "f64": 1e-12}
RDT = {"f32": torch.float32, "f64": torch.float64}


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("nx", [576, 648, 768, 864, 972, 1024])
def test_long_real_rows(nx, dt, offset):
    from paper_1509_07685_amd import dks
    ny, nz = 9, 3
    x = np.random.default_rng(nx).standard_normal((1, nz, ny, nx))
    plan = dks.FFTPlan((nx, ny, nz), 1, "r2c", dt)

    def shifted():
        return torch.zeros(x.size + 1, dtype=RDT[dt], device="cuda")[offset:offset + x.size].view(x.shape)

    xd, back = shifted(), shifted()
    xd.copy_(torch.from_numpy(x))
    H = plan.forward(xd)
    plan.inverse(H, out=back)
    torch.cuda.synchronize()
    xq = xd.cpu().numpy().astype(np.float64)
    assert rel_l2(H.cpu().numpy().astype(np.complex128), fo.rdft3(xq)) <= TOL[dt]
    Hq = H.cpu().numpy().astype(np.complex128)
    assert rel_l2(back.cpu().numpy().astype(np.float64), fo.irdft3(Hq, nx)) <= TOL[dt]
