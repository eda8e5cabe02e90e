"""D2Q9 runs where windows or tiles hold no fluid, and at the most steps per
launch: the bits of single steps."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


def _compare(torch, m, periodic, counts, storage, model="quasi-compressible", collision="bgk"):
    t = lbm.Tiles(m, (16, 16, 1), periodic)
    kw = dict(lattice=9, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), model=model, collision=collision)
    rng = np.random.default_rng(1)
    rho = torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, m.shape)))
    one, run = lbm.Solver(t, **kw), lbm.Solver(t, **kw)
    one.init(rho)
    run.init(rho)
    for n in counts:
        run.step(n)
        for _ in range(n):
            one.step()
        assert torch.equal(run.pdfs_export(), one.pdfs_export()), n


@pytest.mark.parametrize("edge,fluid", [(96, 48), (400, 190), (400, 330)])
@pytest.mark.parametrize("corner", [(0, 0), (1, 1)])
@pytest.mark.parametrize("periodic", [0, 3])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_empty_windows(edge, fluid, corner, periodic, storage):
    """Fluid in one corner alone: tiles that are not stored, and windows without a fluid node."""
    import torch
    assert torch.cuda.is_available()
    m = np.ones((1, edge, edge), bool)
    y, x = [c * (edge - fluid) for c in corner]
    m[0, y:y + fluid, x:x + fluid] = np.random.default_rng(edge).random((fluid, fluid)) < 0.2
    _compare(torch, m, periodic, (5, 9, 12), storage)


# windows of 12 and 14 nodes (ten and nine steps) exactly, one short and one over; four and five steps on larger grids
@pytest.mark.parametrize("shape,periodic", [((1, 12, 12), 0), ((1, 13, 24), 0), ((1, 14, 15), 0), ((1, 28, 27), 0),
                                            ((1, 64, 48), 1), ((1, 192, 176), 3), ((1, 400, 416), 3)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("model", ["quasi-compressible", "incompressible"])
@pytest.mark.parametrize("collision", ["bgk", "mrt"])
def test_most_steps(shape, periodic, storage, model, collision):
    import torch
    assert torch.cuda.is_available()
    m = np.random.default_rng(shape[1]).random(shape) < 0.25
    _compare(torch, m, periodic, (4, 9, 10, 19, 20, 30), storage, model, collision)


@pytest.mark.parametrize("tiles", [2, 4, 6, 12])
def test_few_tiles_on_a_small_grid(tiles):
    """192x192 with tiles**2 of 144 tiles stored: as many steps per launch as there are wavefronts for windows."""
    import torch
    assert torch.cuda.is_available()
    m = np.ones((1, 192, 192), bool)
    m[0, :16 * tiles, :16 * tiles] = np.random.default_rng(tiles).random((16 * tiles, 16 * tiles)) < 0.2
    _compare(torch, m, 0, (10, 17, 20), "f64")
