"""The two-pass register FFT on every pair of radices that its table of
factorisations holds, along x and y, against the FP64 oracle; the first
lengths past its range beside them. Each problem pairs a long lateral axis
with a short one, so work-groups with fewer sequences than they hold (rows and
bins that are no multiple of 8 or 4) are among them.

Tolerances (relative L2): the method's targets, 1e-5 in FP32 and 1e-6 in FP64,
or where it is larger eight times the Kaiser-Bessel window's error estimate
exp(-pi w sqrt(1 - 1/sigma)) (1.3e-5 at sigma 1.25, 5e-7 at 1.5, 2e-8 at 2 for
w = 8; two axes and the largest mode's share of it); a wrong twiddle or index
shows as an error of order one in the modes it touches. Batched and
single-problem images are equal bit for bit.
"""
import sys

import numpy as np
import pytest

import oracle
from oracle.quality import rel_l2
from paper_1510_01078_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (oversampled length, oversampling that gives it from an even axis)
LENGTHS = [(8, 2.0), (12, 1.5), (16, 2.0), (18, 1.5), (20, 2.0), (24, 2.0), (30, 1.5), (32, 2.0), (36, 1.5), (40, 2.0),
           (48, 2.0), (50, 1.25), (54, 1.5), (60, 1.5), (64, 2.0), (72, 2.0), (80, 2.0), (90, 1.5), (96, 2.0),
           (100, 1.25), (108, 1.5), (120, 2.0), (128, 2.0), (144, 2.0), (150, 1.5), (160, 2.0), (162, 1.5), (180, 1.5),
           (192, 2.0), (200, 2.0), (216, 2.0), (240, 2.0), (250, 1.25), (256, 2.0), (270, 1.5), (288, 2.0), (300, 1.5),
           (320, 2.0), (324, 1.5), (360, 2.0), (384, 2.0), (400, 2.0), (432, 2.0), (450, 1.5), (480, 2.0), (486, 1.5),
           (500, 2.0), (512, 2.0), (540, 1.5), (576, 2.0), (600, 2.0), (640, 2.0), (648, 1.5), (720, 2.0)]


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def _pairs():
    """Along x a length of the list, along y the one opposite it among those
    of the same oversampling."""
    out = []
    for s in sorted({s for _, s in LENGTHS}):
        ns = [n for n, t in LENGTHS if t == s]
        out += [(n, ns[len(ns) - 1 - i], s) for i, n in enumerate(ns)]
    return out


def _problem(nx_over, ny_over, sigma, nz=4):
    rng = np.random.default_rng(nx_over * 1000 + ny_over)
    shape = (round(nx_over / sigma), round(ny_over / sigma), nz)
    ext = (shape[0] * 0.25e-3, shape[1] * 0.25e-3, max(2e-3, nz * 0.25e-3))
    return inputs.random_problem(rng, 37, 45, shape, ext, dt=30e-9)


def _kw(sigma):
    return dict(kernel="kaiser_bessel", sigma_xy=sigma, width_xy=8, sigma_t=2.0, width_t=8)


@pytest.mark.parametrize("nx_over,ny_over,sigma", _pairs())
def test_lengths_vs_oracle(dev, nx_over, ny_over, sigma):
    from paper_1510_01078_amd import Plan
    p = _problem(nx_over, ny_over, sigma)
    ref = oracle.reconstruct(p.xy, p.h, p.g, p.dt, p.c, p.shape, p.extent)
    for precision, tol in (("fp32", 1e-5), ("fp64", 1e-6)):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision=precision, **_kw(sigma))
        assert pl.info["nx_over"] == nx_over and pl.info["ny_over"] == ny_over
        err = rel_l2(pl.reconstruct(torch.from_numpy(p.g).to(dev, pl.dtype)).cpu().numpy().astype(np.float64), ref)
        pl.close()
        _say(f"[gpu] lengths {nx_over} x {ny_over} {precision}: {err:.2e}")
        assert err <= max(tol, 8 * np.exp(-np.pi * 8 * np.sqrt(1 - 1 / sigma)))


@pytest.mark.parametrize("nx,ny,nz", [(4, 6, 640), (6, 4, 576), (10, 8, 486), (8, 12, 384), (640, 4, 16), (4, 640, 36),
                                      (486, 6, 250), (6, 500, 8), (720, 4, 6), (4, 720, 10), (6, 8, 720), (288, 18, 90),
                                      (18, 288, 162), (320, 20, 288), (20, 320, 400), (54, 50, 54)])
def test_image_lengths_vs_oracle(dev, nx, ny, nz):
    """The image's own transforms (gather's x pass, y pass, complex-to-real z
    pass): each class of lengths per axis, z runs that are no multiple of a
    group's 8 or 16 modes, the longest and the first past the range."""
    from paper_1510_01078_amd import Plan
    p = _problem(2 * nx, 2 * ny, 2.0, nz)
    ref = oracle.reconstruct(p.xy, p.h, p.g, p.dt, p.c, p.shape, p.extent)
    for precision, tol in (("fp32", 1e-5), ("fp64", 1e-6)):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision=precision, **_kw(2.0))
        err = rel_l2(pl.reconstruct(torch.from_numpy(p.g).to(dev, pl.dtype)).cpu().numpy().astype(np.float64), ref)
        pl.close()
        _say(f"[gpu] image {nx} x {ny} x {nz} {precision}: {err:.2e}")
        assert err <= tol


@pytest.mark.parametrize("nx,ny,nz,width", [(8, 6, 4, 8), (24, 40, 6, 8), (48, 18, 4, 2), (96, 20, 4, 8), (100, 30, 6, 12),
                                            (20, 100, 4, 10), (144, 12, 4, 8), (160, 16, 4, 6), (192, 16, 4, 8),
                                            (192, 4, 4, 8), (216, 10, 4, 12), (240, 10, 4, 8), (256, 36, 4, 8),
                                            (320, 8, 4, 8), (16, 360, 4, 8)])
def test_forward_lengths_vs_oracle(dev, nx, ny, nz, width):
    """The forward model's transposed lateral transforms: every class of the
    fused x transform and interpolation, strips of one and two home-tile rows,
    short y axes that the strip wraps around, narrow and wide footprints, and
    lengths whose second pass has more butterflies than threads (passes in LDS
    then). The adjoint beside it: <A f, g> = <f, A* g> within the FP32 sums'
    rounding (1e-5 of the norms' product)."""
    from oracle import forward_model as fm
    from paper_1510_01078_amd import Plan
    p = _problem(2 * nx, 2 * ny, 2.0, nz)
    rng = np.random.default_rng(nx + ny)
    f = rng.standard_normal(p.shape)
    ref = fm.forward(f, p.xy, p.nt, p.dt, p.c, p.extent)
    kw = dict(_kw(2.0), width_xy=width)
    tol = max(1e-5, 8 * np.exp(-np.pi * width * np.sqrt(0.5)))
    pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision="fp32", **kw)
    fd = torch.from_numpy(f).to(dev, torch.float32)
    gd = torch.from_numpy(p.g).to(dev, torch.float32)
    a, b = pl.forward(fd), pl.adjoint(gd)
    err = rel_l2(a.cpu().numpy().astype(np.float64), ref)
    gap = abs(float((a.double() * gd.double()).sum()) - float((fd.double() * b.double()).sum()))
    scale = float(a.double().norm() * gd.double().norm())
    pl.close()
    _say(f"[gpu] forward {nx} x {ny} x {nz} w {width}: {err:.2e}, adjointness {gap / scale:.1e}")
    assert err <= tol and gap <= 1e-5 * scale


@pytest.mark.parametrize("nx,ny,nz", [(54, 50, 54), (8, 18, 128), (20, 16, 400), (288, 6, 30), (16, 162, 10),
                                      (320, 20, 20), (6, 8, 640), (4, 6, 648)])
def test_forward_image_lengths_vs_oracle(dev, nx, ny, nz):
    """The forward model's transforms of the image: each class per axis, rows
    that are no multiple of a group's, a z length with a compile-time form, the
    longest z rows and the first past the range."""
    from oracle import forward_model as fm
    from paper_1510_01078_amd import Plan
    p = _problem(2 * nx, 2 * ny, 2.0, nz)
    f = np.random.default_rng(nx + nz).standard_normal(p.shape)
    ref = fm.forward(f, p.xy, p.nt, p.dt, p.c, p.extent)
    for precision, tol in (("fp32", 1e-5), ("fp64", 1e-6)):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision=precision, **_kw(2.0))
        err = rel_l2(pl.forward(torch.from_numpy(f).to(dev, pl.dtype)).cpu().numpy().astype(np.float64), ref)
        pl.close()
        _say(f"[gpu] forward image {nx} x {ny} x {nz} {precision}: {err:.2e}")
        assert err <= tol


def test_batch_of_all_classes_equals_single(dev):
    from paper_1510_01078_amd import Plan
    from paper_1510_01078_amd.batch import Batch, problem_dict
    probs = [_problem(n, m, 2.0, z) for n, m, z in ((64, 96, 54), (256, 40, 288), (320, 60, 400), (40, 384, 4),
                                                    (480, 512, 6), (640, 20, 720), (720, 64, 90), (1152, 12, 8))]
    b = Batch([problem_dict(p) for p in probs], precision="fp32", defaults=_kw(2.0))
    gs = [torch.from_numpy(p.g).to(dev, torch.float32) for p in probs]
    outs = b.reconstruct(gs)
    torch.cuda.synchronize()
    same = []
    for p, g, o in zip(probs, gs, outs):
        pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision="fp32", **_kw(2.0))
        same.append(bool(torch.equal(pl.reconstruct(g), o)))
        pl.close()
    b.close()
    _say(f"[gpu] batch of every length class vs single plans bitwise: {same}")
    assert all(same)
