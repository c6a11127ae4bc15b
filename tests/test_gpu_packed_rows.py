"""The second row layout of the intermediate arrays: a plan that fits the
allocation-free call's scratch only without the padding to 128-byte lines keeps
packed rows (here 54-point grid rows, 600-point columns and an odd number of
half lines of band bins), for every call. All of them on such a plan: against
the FP64 oracle within 1e-5 (the FP32 bound), the allocation-free call and a
batch bit for bit equal to the plain call."""
import sys

import numpy as np
import pytest

import oracle
from oracle import forward_model as fm
from oracle.quality import rel_l2
from paper_1510_01078_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KW = dict(kernel="kaiser_bessel", sigma_xy=1.5, width_xy=8, sigma_t=2.0, width_t=8)


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _workspace(m, shape, info, unit):
    """Bytes of the three regions with rows of a multiple of `unit` values."""
    up = lambda n: -(-n // unit) * unit
    region = lambda *sizes: -(-max(sizes) * 8 // 256) * 256
    nx, ny, nz = shape
    nxo, nyo, nb = info["nx_over"], info["ny_over"], info["band_bins"]
    return (region(nb * nyo * up(nxo), nx * ny * up(nb)) + region(nb * nx * up(nyo), nx * ny * max(up(nz // 2), nz // 2 + 1))
            + region(m * up(nb)))


def test_packed_rows():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_01078_amd import Plan
    from paper_1510_01078_amd import _native as N
    from paper_1510_01078_amd.batch import Batch, problem_dict
    dev = torch.device("cuda", 0)
    shape = (36, 400, 8)
    rng = np.random.default_rng(3)
    p = inputs.random_problem(rng, 37, 750, shape, tuple(n * 0.25e-3 for n in shape), dt=83e-9)
    f = rng.standard_normal(shape)
    pl = Plan(p.xy, p.nt, p.dt, p.c, p.shape, p.extent, sensor_h=p.h, precision="fp32", **KW)
    packed, padded = (_workspace(p.m, shape, pl.info, u) for u in (1, 16))
    _say(f"[gpu] {pl.info['nx_over']} x {pl.info['ny_over']} x {pl.info['band_bins']} bins: {pl.info['workspace_bytes']} "
         f"bytes, packed {packed}, padded {padded}")
    assert packed <= N.PAT_NOALLOC_SCRATCH_BYTES < padded
    assert pl.info["workspace_bytes"] == packed
    g = torch.from_numpy(p.g).to(dev, torch.float32)
    fd = torch.from_numpy(f).to(dev, torch.float32)
    img = pl.reconstruct(g)
    out = torch.full(shape, float("nan"), dtype=torch.float32, device=dev)
    pl.reconstruct_noalloc(g, out)
    torch.cuda.synchronize()
    assert torch.equal(img, out)
    num = lambda t: t.cpu().numpy().astype(np.float64)
    e = {"image": rel_l2(num(img), oracle.reconstruct(p.xy, p.h, p.g, p.dt, p.c, p.shape, p.extent)),
         "adjoint": rel_l2(num(pl.adjoint(g)), fm.adjoint(p.g, p.xy, p.dt, p.c, p.shape, p.extent)),
         "model": rel_l2(num(pl.forward(fd)), fm.forward(f, p.xy, p.nt, p.dt, p.c, p.extent))}
    for a in (0, 1):
        e["xy"[a]] = rel_l2(num(pl.forward_dxy(fd, a)), fm.forward(f, p.xy, p.nt, p.dt, p.c, p.extent, deriv="xy"[a]))
    b = Batch([problem_dict(p)], precision="fp32", defaults=KW)
    same = bool(torch.equal(b.reconstruct([g])[0], img))
    b.close()
    pl.close()
    _say(f"[gpu] packed rows vs oracle: {e}, batch equal {same}")
    assert max(e.values()) <= 1e-5 and same
