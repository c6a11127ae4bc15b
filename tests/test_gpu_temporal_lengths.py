"""The temporal FFT's register form against the FP64 oracle: two and three
passes of every class of radices, the largest length, the one length in range
that keeps its passes in LDS (6250 = 10 25 25), an odd sensor count (the last
work-group holds one sensor), and enough sensors that a work-group takes two
and four pairs. Reconstruction (weighted traces) and adjoint (unit weights).

Tolerances: 1e-5 in FP32 and 1e-6 in FP64 (relative L2), the method's targets;
a wrong twiddle or slot shows as an error of order one in the bins it touches.
Batched and single-problem images are equal bit for bit.
"""
import sys

import numpy as np
import pytest

import oracle
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


def _problem(nt_over, m):
    rng = np.random.default_rng(nt_over + m)
    nt = nt_over // 2
    # the trace spans a few periods of the depth whatever its length
    return inputs.random_problem(rng, m, nt, (8, 6, 8), (2e-3, 1.5e-3, 2e-3), dt=min(60e-9, 20e-6 / nt))


@pytest.mark.parametrize("nt_over,m", [(128, 7), (300, 5), (480, 6), (640, 5), (648, 5), (720, 4), (1250, 5), (1280, 3),
                                       (1458, 5), (1920, 2), (2048, 5), (2500, 5), (2560, 7), (3200, 5), (4096, 3),
                                       (4374, 5), (5000, 3), (6250, 5), (7776, 3), (8000, 2), (8192, 5),
                                       (64, 4097), (100, 8195)])
def test_lengths_vs_oracle(dev, nt_over, m):
    from paper_1510_01078_amd import Plan
    p = _problem(nt_over, m)
    ref = oracle.reconstruct(p.xy, p.h, p.g, p.dt, p.c, p.shape, p.extent)
    ref_a = fm.adjoint(p.g, p.xy, p.dt, p.c, p.shape, p.extent)
    for precision, tol in (("fp32", 1e-5), ("fp64", 1e-6)):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision=precision, **KW)
        assert pl.info["nt_over"] == nt_over
        g = torch.from_numpy(p.g).to(dev, pl.dtype)
        e_r = rel_l2(pl.reconstruct(g).cpu().numpy().astype(np.float64), ref)
        e_a = rel_l2(pl.adjoint(g).cpu().numpy().astype(np.float64), ref_a)
        pl.close()
        _say(f"[gpu] temporal {nt_over} x {m} sensors {precision}: {e_r:.2e}, adjoint {e_a:.2e}")
        assert e_r <= tol and e_a <= tol


def test_batch_equals_single(dev):
    from paper_1510_01078_amd import Plan
    from paper_1510_01078_amd.batch import Batch, problem_dict
    probs = [_problem(n, m) for n, m in ((128, 7), (300, 5), (480, 2051), (720, 5), (2560, 4), (3200, 5), (5000, 3),
                                         (6250, 3), (8192, 2))]
    b = Batch([problem_dict(p) for p in probs], precision="fp32", defaults=KW)
    gs = [torch.from_numpy(p.g).to(dev, torch.float32) for p in probs]
    outs = b.reconstruct(gs)
    torch.cuda.synchronize()
    same = []
    for p, g, o in zip(probs, gs, outs):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision="fp32", **KW)
        same.append(bool(torch.equal(pl.reconstruct(g), o)))
        pl.close()
    b.close()
    _say(f"[gpu] batch of temporal lengths vs single plans bitwise: {same}")
    assert all(same)
