"""Several D2Q9 steps in one launch: the state is that of single steps, at the
edges of the windows, over walls and periodic axes, with leftovers of every
length and inside graphs."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


# small grids (eight steps a launch) with windows of 16 exactly, one short and one over; a larger one (four steps)
SHAPES = [((1, 1, 1), 0), ((1, 7, 5), 0), ((1, 16, 16), 3), ((1, 17, 33), 0), ((1, 64, 48), 1), ((1, 31, 80), 1),
          ((1, 270, 289), 0), ((1, 288, 272), 3)]


@pytest.mark.parametrize("shape,periodic", SHAPES)
@pytest.mark.parametrize("storage,eps", [("f64", 2.0 ** -53), ("f32", 2.0 ** -24)])
@pytest.mark.parametrize("model", ["quasi-compressible", "incompressible"])
@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("graph_steps", [0, 11])
def test_runs_of_steps_are_single_steps(torch, shape, periodic, storage, eps, model, collision, graph_steps):
    """BGK spells out each rounding, so its bits agree; MRT leaves contractions to
    the compiler: per step at most 100 roundings of values of order 1."""
    rng = np.random.default_rng(shape[1] * 1000 + shape[2])
    m = rng.random(shape) < 0.25
    m.flat[0] = False
    t = lbm.Tiles(m, (16, 16, 1), periodic)
    kw = dict(lattice=9, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), model=model, collision=collision)
    rho = torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape)))
    one, run = lbm.Solver(t, **kw), lbm.Solver(t, graph_steps=graph_steps, **kw)
    one.init(rho)
    run.init(rho)
    steps = 0
    for n in (1, 2, 3, 8, 11, 14):
        run.step(n)
        for _ in range(n):
            one.step(1)
        steps += n
        a, b = run.pdfs_export(), one.pdfs_export()
        d = float((a - b).abs().max())
        assert d <= (0.0 if collision == "bgk" else 100 * steps * eps)
    assert run.step_count == one.step_count == steps
