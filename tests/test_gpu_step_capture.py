"""Steps captured by the caller: an even number of steps ends in the copy it
starts from, so the caller's graph can be replayed, with steps outside it in
between, whatever number of launches the steps take."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tile", [((1, 48, 64), (16, 16, 1)), ((1, 288, 272), (16, 16, 1)),
                                        ((8, 12, 16), (4, 4, 4))])
@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("pattern", ["two-copy", "single-copy"])
@pytest.mark.parametrize("steps", [2, 4, 6, 10, 26])
def test_replays_of_a_callers_graph(shape, tile, storage, pattern, steps):
    import torch
    assert torch.cuda.is_available()
    m = np.random.default_rng(steps).random(shape) < 0.25
    t = lbm.Tiles(m, tile, 0)
    kw = dict(lattice=9 if tile[2] == 1 else 19, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern)
    side = torch.cuda.Stream()
    run, one = lbm.Solver(t, stream=side, **kw), lbm.Solver(t, **kw)
    run.init()
    one.init()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run.step(steps)
    for k in range(4):
        with torch.cuda.stream(side):
            graph.replay()
            run.step(4 * k)  # an even number of steps of its own between the replays
        side.synchronize()
        for _ in range(steps + 4 * k):
            one.step()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            a = run.pdfs_export()
        side.synchronize()
        assert torch.equal(a, one.pdfs_export())
