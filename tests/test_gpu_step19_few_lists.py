"""Steps of few tiles from a list and on the persistent grid store directly,
those of more through LDS: the same bits on both sides of each line."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


# tiles: 64 nx / 32 in FP64 and 64 nx / 16 in FP32, and one more sample of one tile
@pytest.mark.parametrize("storage,nz,nx", [("f64", 8, 5), ("f64", 8, 63), ("f64", 8, 65), ("f64", 8, 255),
                                           ("f64", 8, 257), ("f32", 16, 5), ("f32", 16, 255), ("f32", 16, 257)])
@pytest.mark.parametrize("pattern", ["two-copy", "single-copy"])
@pytest.mark.parametrize("model", ["quasi-compressible", "incompressible"])
def test_lists_on_both_sides(storage, nz, nx, pattern, model):
    import torch
    assert torch.cuda.is_available()
    shape = (nz, 64, nx)
    rng = np.random.default_rng(nx)
    m = rng.random(shape) < 0.2
    t = lbm.Tiles(m, (4, 4, 4), 0)
    rho = torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape)))
    kw = dict(lattice=19, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern, model=model)
    one = lbm.Solver(t, step_kernel="scalar", **kw)
    one.init(rho)
    one.step(6)
    want = one.pdfs_export().flatten()
    two = lbm.Tiles.concat([t, lbm.Tiles(np.zeros((4, 4, 4), bool))])
    for persistent in (0, 1):
        s = lbm.Solver(two, persistent=persistent, **kw)
        s.init(torch.cat([rho.flatten(), torch.ones(64, dtype=torch.float64)]))
        s.set_active([1, 0])
        s.step(6)
        assert torch.equal(s.pdfs_export().flatten()[:want.numel()], want)
