"""The batched launches on every kernel variant (classes of FFT lengths,
numbers of temporal passes, lengths with their passes in LDS): a persistent
grid of few work-groups, each looping over items of several problems and
reusing its LDS, gives the bits of the default launch (one work-group per
item), and the default call captured in a HIP graph gives, on every replay,
those of the eager call."""
import sys

import numpy as np
import pytest

from paper_1510_01078_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KW = dict(kernel="kaiser_bessel", sigma_xy=2.0, width_xy=8, sigma_t=2.0, width_t=8)

# (image, samples): lateral lengths of the classes up to 16, 20 and 32 and past
# 640 points, image lengths likewise, temporal lengths of two and three passes,
# with the first pass in rounds (3200) and without factors (6250)
PROBLEMS = [((64, 96, 54), 64), ((20, 18, 16), 150), ((40, 18, 30), 240), ((18, 288, 12), 360), ((320, 6, 20), 1280),
            ((6, 20, 400), 1600), ((8, 360, 6), 2500), ((720, 4, 6), 3125), ((4, 12, 720), 4096)]


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", params=["fp32", "fp64"])
def setup(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1510_01078_amd.batch import Batch, problem_dict
    probs = []
    for i, (shape, nt) in enumerate(PROBLEMS):
        ext = tuple(max(2e-3, n * 0.25e-3) for n in shape)
        probs.append(inputs.random_problem(np.random.default_rng(i), 21 + 2 * i, nt, shape, ext, dt=min(30e-9, 20e-6 / nt)))
    b = Batch([problem_dict(p) for p in probs], precision=request.param, defaults=KW)
    gs = [torch.from_numpy(p.g).to("cuda", b.dtype) for p in probs]
    yield b, gs
    b.close()


def test_small_persistent_grids_same_bits(setup):
    b, gs = setup
    ref = [o.clone() for o in b.reconstruct(gs)]
    assert all(bool(torch.isfinite(o).all()) and float(o.abs().max()) > 0 for o in ref)
    for blocks in (1, 24, 512):
        b.set_grid(blocks)
        got = [o.clone() for o in b.reconstruct(gs)]
        torch.cuda.synchronize()
        same = [bool(torch.equal(x, y)) for x, y in zip(ref, got)]
        _say(f"[gpu] {b.precision} grid of {blocks}: equal to one work-group per item {same}")
        b.set_grid(0)
        assert all(same)


def test_default_grid_graph_replays(setup):
    b, gs = setup
    static_in = [g.clone() for g in gs]
    static_out = [torch.empty(s, dtype=b.dtype, device="cuda") for s in b.shapes]
    b.reconstruct(static_in, static_out)  # warm-up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.reconstruct(static_in, static_out)
    torch.cuda.synchronize()
    for r in range(3):
        for s_in, g in zip(static_in, gs):
            s_in.copy_(g * (1.0 + 0.5 * r))
        torch.cuda.synchronize()
        eager = [o.clone() for o in b.reconstruct([s.clone() for s in static_in])]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        same = [bool(torch.equal(x, y)) for x, y in zip(eager, static_out)]
        _say(f"[gpu] {b.precision} graph replay {r}: equal to eager {same}")
        assert all(same)
