"""The position derivatives (pat_forward_dxy) keep their passes in LDS at every
length: the compile-time lengths of the image's transforms (128, 192, 256, 512
along x, y and z) and of the lateral ones (256, 288, 384, 512), the runtime
plan beside them, and the transposed y pass where its work-groups hold six or
seven bins (540 to 640 points) or one (1024), each against the FP64 oracle.

Tolerances (relative L2): 1e-5 in FP32 and 1e-6 in FP64, the bounds of the
derivatives at this window setting (sigma 2, Kaiser-Bessel w 8, whose own error
is about 1e-7); a wrong twiddle, bin or mode shows as an error of order one.
"""
import sys

import numpy as np
import pytest

from oracle import forward_model as fm
from oracle.quality import rel_l2
from paper_1510_01078_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KW = dict(kernel="kaiser_bessel", sigma_xy=2.0, width_xy=8, sigma_t=2.0, width_t=8)


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


@pytest.mark.parametrize("shape", [(128, 4, 8), (256, 4, 8), (192, 6, 4), (144, 4, 4), (512, 4, 4),
                                   (8, 128, 4), (8, 192, 6), (8, 144, 4), (6, 256, 4), (6, 512, 8),
                                   (6, 4, 128), (4, 6, 192), (4, 4, 256), (4, 4, 512), (6, 10, 150),
                                   (8, 270, 4), (10, 288, 4), (8, 300, 6), (12, 320, 4), (30, 20, 12)])
def test_derivatives_vs_oracle(dev, shape):
    from paper_1510_01078_amd import Plan
    rng = np.random.default_rng(sum(shape))
    ext = (shape[0] * 0.25e-3, shape[1] * 0.25e-3, max(2e-3, shape[2] * 0.25e-3))
    p = inputs.random_problem(rng, 37, 64, shape, ext, dt=30e-9)
    f = rng.standard_normal(shape)
    ref = [fm.forward(f, p.xy, p.nt, p.dt, p.c, p.extent, deriv=a) for a in "xy"]
    for precision, tol in (("fp32", 1e-5), ("fp64", 1e-6)):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision=precision, **KW)
        fd = torch.from_numpy(f).to(dev, pl.dtype)
        err = [rel_l2(pl.forward_dxy(fd, a).cpu().numpy().astype(np.float64), ref[a]) for a in (0, 1)]
        info = {k: pl.info[k] for k in ("nx_over", "ny_over", "forward_fused")}
        pl.close()
        _say(f"[gpu] derivatives {shape} {precision} {info}: {err[0]:.2e} {err[1]:.2e}")
        assert max(err) <= tol
